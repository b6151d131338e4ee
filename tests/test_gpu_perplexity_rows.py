"""Perplexity calibration of more rows than one launch takes at 64 threads a row
(2^26 and a few): rows of every launch against the oracle to 1e-9.
"""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


def test_rows():
    from paper_1611_02568_amd import pixelsne
    n, k, u = (1 << 26) + 5, 2, 1.5
    d2 = torch.rand(n, k, dtype=torch.float64, device="cuda",
                    generator=torch.Generator(device="cuda").manual_seed(1))
    P, beta = pixelsne.perplexity(d2, u)
    at = np.concatenate([[0, (1 << 22) - 1, 1 << 22, (1 << 26) - 1], np.arange(1 << 26, n),
                         np.random.default_rng(2).choice(n, 500, replace=False)])
    rows = torch.as_tensor(at, device="cuda")
    oP, ob, _ = oracle.perplexity(d2[rows].cpu().numpy(), u)
    np.testing.assert_allclose(P[rows].cpu().numpy(), oP, rtol=1e-9, atol=0)
    np.testing.assert_allclose(beta[rows].cpu().numpy(), ob, rtol=1e-9, atol=0)
