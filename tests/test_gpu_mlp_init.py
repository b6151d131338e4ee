"""The network's initial weights: those of a C++ program that draws them from the
standard library's generator and distribution, layer by layer, bit for bit.
"""
import subprocess

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SOURCE = r"""
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <random>
int main(int, char** v) {
    const long size[4] = {atol(v[2]), atol(v[3]), atol(v[4]), 2};
    std::mt19937_64 rng(strtoull(v[1], nullptr, 10));
    std::normal_distribution<float> nd(0.f, 1.f);
    for (int l = 0; l < 3; l++) {
        const float sc = sqrtf(2.f / (float)size[l]);
        for (long i = 0; i < size[l] * size[l + 1]; i++) {
            const float w = nd(rng) * sc;
            fwrite(&w, 4, 1, stdout);
        }
        const float zero = 0.f;
        for (long i = 0; i < size[l + 1]; i++) fwrite(&zero, 4, 1, stdout);
    }
}
"""


@pytest.mark.parametrize("d,h1,h2,seed", [(1, 1, 1, 0), (5, 7, 3, 11), (100, 256, 129, 2 ** 63 + 5)])
def test_weights(tmp_path, d, h1, h2, seed):
    from paper_1611_02568_amd import pixelsne
    src, exe = tmp_path / "w.cpp", tmp_path / "w"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-O1", "-std=c++17", str(src), "-o", str(exe)], check=True)
    want = np.frombuffer(subprocess.run([str(exe), str(seed), str(d), str(h1), str(h2)], check=True,
                                        capture_output=True).stdout, np.float32)
    net = pixelsne.MLP(d, h1, h2, seed=seed)
    assert np.array_equal(net.params().cpu().numpy(), want)
