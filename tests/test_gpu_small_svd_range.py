"""The small SVD near the end of FP64's range: with S scaled by a power of two every
step scales exactly, so modes, singular values and coefficients keep their bits as
long as no sum of the algorithm overflows: the squares of the columns' squared
norms, sigma_1^4, at sigma_1 = 2^255.9 the largest of them."""

import numpy as np
import pytest
import torch

import synth
from test_gpu_parity import run_gpu, upload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("l", [8, 16, 30, 60, 128])
def test_scaled(l):
    m, n = 600, 300
    St = synth.lowrank_exp(m, n, decay=0.05, noise_std=1e-6, seed=l)["St"]
    St = St * (2.0 ** -0.1 / np.linalg.norm(St, 2))
    print(f"[case] l={l}", flush=True)
    ref, got = (run_gpu(upload(St * s, torch.float64)[0], m, n, l, 0, 1, 5, torch.float64) for s in (1.0, 2.0 ** 256))
    assert np.array_equal(got[0], ref[0])
    assert np.array_equal(got[1], ref[1] * 2.0 ** 256) and np.array_equal(got[2], ref[2] * 2.0 ** 256)
