// What the Barnes-Hut walks of the quadtree and the octree share: a stack of
// sibling groups in lane registers, and the walk of 64 points' union list by
// several wavefronts.
#pragma once

#include "common.h"

namespace psne {
namespace {

// Write a stack entry (four wave-uniform words, in scalar registers) into
// lane `sel` of the four per-lane stack registers.  With one scalar operand
// per vector instruction the lane select goes through m0 (an input operand:
// the compiler writes it with a scalar move); the s_nop adds two wait states
// before it is read.
__device__ __forceinline__ void push_entry(int& a, int& b, int& c, int& d, int va, int vb,
                                           int vc, int vd, int sel) {
    asm("s_nop 1\n\t"
        "v_writelane_b32 %0, %4, m0\n\t"
        "v_writelane_b32 %1, %5, m0\n\t"
        "v_writelane_b32 %2, %6, m0\n\t"
        "v_writelane_b32 %3, %7, m0"
        : "+v"(a), "+v"(b), "+v"(c), "+v"(d)
        : "s"(va), "s"(vb), "s"(vc), "s"(vd), "{m0}"(sel));
}

// The traversal's stack: entry k (a sibling group: its first cell, size and
// level, and the 64-bit mask of lanes that descend into it) lives in lane k of
// four registers.  A walk pushes at most three pending groups per level plus
// the one it expands next, so 3 (levels) + 1 entries suffice: 52 for the pixel
// tree (at most 17 levels), 100 for the data-driven tree (33 levels), which
// takes a second set of four registers for entries 64..127 (DEEP), as does the
// octree (at most seven pending per level, 11 levels).
template <bool DEEP>
struct WaveStack {
    int f0 = 0, i0 = 0, lo0 = 0, hi0 = 0;
    int f1 = 0, i1 = 0, lo1 = 0, hi1 = 0;
    __device__ __forceinline__ void push(int sp, int f, int info, int lo, int hi) {
        if (!DEEP || sp < kWave) push_entry(f0, i0, lo0, hi0, f, info, lo, hi, sp);
        else push_entry(f1, i1, lo1, hi1, f, info, lo, hi, sp - kWave);
    }
    __device__ __forceinline__ void read(int sp, uint32_t& first, uint32_t& info,
                                         uint64_t& mask) const {
        if (!DEEP || sp < kWave) {
            first = (uint32_t)__builtin_amdgcn_readlane(f0, sp);
            info = (uint32_t)__builtin_amdgcn_readlane(i0, sp);
            mask = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane(hi0, sp) << 32) |
                   (uint64_t)(uint32_t)__builtin_amdgcn_readlane(lo0, sp);
        } else {
            const int k = sp - kWave;
            first = (uint32_t)__builtin_amdgcn_readlane(f1, k);
            info = (uint32_t)__builtin_amdgcn_readlane(i1, k);
            mask = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane(hi1, k) << 32) |
                   (uint64_t)(uint32_t)__builtin_amdgcn_readlane(lo1, k);
        }
    }
};

// A sibling group in one word: its first cell and its size, 1 to 4 (as
// Node::child holds a cell's children).
__device__ __forceinline__ uint32_t group_first(uint32_t g) { return g & 0x3FFFFFFFu; }
__device__ __forceinline__ uint32_t group_num(uint32_t g) { return (g >> 30) + 1u; }

// The groups of two levels, one segment of CAP per wavefront.
template <int G, int CAP>
struct WalkLists {
    uint64_t mask[2][G][CAP];
    uint32_t group[2][G][CAP];
    uint32_t num[2][G];
};

constexpr int kWalkFlush = 8;     // groups gathered in registers before they go to LDS

// The union list of 64 points (ALL: the lanes that hold one) walked by the G
// wavefronts of a block, each of which holds all 64 points in WK.  The list is
// walked level by level: the sibling groups of a level lie in LDS, wavefront W
// takes the groups W, W + G, ..., and appends the groups that its lanes open
// to its own segment of the next level, so which wavefront meets a cell, and
// the order of every lane's partial sums, depend on the tree alone.  Known
// groups are loaded one ahead of their use (AHEAD), where a depth-first walk
// waits for each group's records.  A segment that is full sends its wavefront down
// depth first instead (theta near 0 opens whole levels): at most kWalkFlush +
// 7 groups are then pending and each of the at most 17 levels of the quadtree
// adds at most three (11 levels and seven for the octree, DEEP), which the
// stack holds.
template <int G, int CAP, bool DEEP, bool AHEAD = true, typename W>
__device__ __forceinline__ void walk_shared(W& wk, WalkLists<G, CAP>& l, int w, uint64_t all) {
    const int lane = lane_id();
    if (threadIdx.x < G) l.num[0][threadIdx.x] = threadIdx.x == 0 && all ? 1u : 0u;
    if (threadIdx.x == 0) {
        l.mask[0][0][0] = all;
        l.group[0][0][0] = 0u;                       // the root: cell 0, one cell
    }
    __syncthreads();
    for (int level = 0;; level++) {
        const int b = level & 1;
        // the level's groups in wavefront order: segment starts
        uint32_t start[G + 1];
        start[0] = 0;
        const uint32_t nl = lane < G ? l.num[b][lane < G ? lane : 0] : 0u;
#pragma unroll
        for (int q = 0; q < G; q++)
            start[q + 1] = start[q] + (uint32_t)__builtin_amdgcn_readlane((int)nl, q);
        const uint32_t total = start[G];
        if (total == 0) break;
        WaveStack<DEEP> st;      // groups opened by this wavefront, not yet in LDS
        int sp = 0;
        uint32_t put = 0;        // groups of the next level in this wavefront's segment
        auto push = [&](uint32_t group, int lv, uint64_t om) {
            st.push(sp, (int)group, lv, (int)(uint32_t)om, (int)(uint32_t)(om >> 32));
            sp++;
        };
        auto flush = [&]() {
            if (put + (uint32_t)sp <= (uint32_t)CAP) {
                if (lane < sp) {
                    l.group[b ^ 1][w][put + lane] = (uint32_t)st.f0;
                    l.mask[b ^ 1][w][put + lane] =
                        ((uint64_t)(uint32_t)st.hi0 << 32) | (uint64_t)(uint32_t)st.lo0;
                }
                put += (uint32_t)sp;
                sp = 0;
                return;
            }
            while (sp > 0) {     // no room: the pending groups depth first
                sp--;
                uint32_t group, lv;
                uint64_t mask;
                st.read(sp, group, lv, mask);
                const uint32_t first = group_first(group);
                wk.meet(wk.load(first), first, group_num(group), (int)lv, mask, push);
            }
        };
        // this wavefront's groups, 64 at a time into lanes
        for (uint32_t e0 = (uint32_t)w; e0 < total; e0 += (uint32_t)(G * kWave)) {
            const uint32_t e = e0 + (uint32_t)(G * lane);
            uint32_t group = 0;
            uint64_t mask = 0;
            if (e < total) {
                int seg = 0;
#pragma unroll
                for (int q = 1; q < G; q++) seg += e >= start[q] ? 1 : 0;
                uint32_t at = e;
#pragma unroll
                for (int q = 1; q < G; q++) at = seg == q ? e - start[q] : at;
                group = l.group[b][seg][at];
                mask = l.mask[b][seg][at];
            }
            const int mlo = (int)(uint32_t)mask, mhi = (int)(uint32_t)(mask >> 32);
            const uint32_t left = (total - e0 + (uint32_t)G - 1) / (uint32_t)G;
            const int m = left < (uint32_t)kWave ? (int)left : kWave;
            auto group_at = [&](int k) {
                return (uint32_t)__builtin_amdgcn_readlane((int)group, k);
            };
            auto lanes_at = [&](int k) {
                return ((uint64_t)(uint32_t)__builtin_amdgcn_readlane(mhi, k) << 32) |
                       (uint64_t)(uint32_t)__builtin_amdgcn_readlane(mlo, k);
            };
            if constexpr (AHEAD) {
                uint32_t cur = group_at(0);
                typename W::Group rec = wk.load(group_first(cur));
                for (int k = 0; k < m; k++) {
                    const uint32_t nxt = group_at(k + 1 < m ? k + 1 : k);
                    const typename W::Group rec1 = wk.load(group_first(nxt));
                    wk.meet(rec, group_first(cur), group_num(cur), level, lanes_at(k), push);
                    if (sp >= kWalkFlush) flush();
                    rec = rec1;
                    cur = nxt;
                }
            } else {
                for (int k = 0; k < m; k++) {
                    const uint32_t cur = group_at(k);
                    wk.meet(wk.load(group_first(cur)), group_first(cur), group_num(cur), level,
                            lanes_at(k), push);
                    if (sp >= kWalkFlush) flush();
                }
            }
        }
        if (sp > 0) flush();
        if (lane == 0) l.num[b ^ 1][w] = put;
        __syncthreads();
    }
}

}  // namespace
}  // namespace psne
