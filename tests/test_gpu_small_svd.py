"""The small SVD of step 6 at every padded width: the pivoted Cholesky factor and
the one-sided Jacobi sweeps run on blocks of eight columns, lp / 16 waves per
matrix, so the widths at and around multiples of 8, 16 and 64 are where a pair,
a block or a padded column could be lost. Against the oracle's randomized POD
on the same sketch, with the tolerances of the parity tests (FP64: the factor
route; FP32: the Gram route)."""

import numpy as np
import pytest
import torch

import synth
from test_gpu_parity import case, run_gpu, upload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("l", [1, 8, 16, 17, 32, 41, 48, 63, 64, 65, 80, 96, 105, 112, 121, 128])
def test_every_width(l, dtype):
    g = synth.lowrank_exp(600, 300, decay=0.04, noise_std=1e-5, seed=100 + l)
    case(g["St"], max(1, l - l // 4), l - max(1, l - l // 4), 1, 7 + l, dtype, name=f"l={l}")


@pytest.mark.parametrize("l", [20, 60, 100, 128])
def test_equal_singular_values(l):
    # all singular values of S equal: every pair of columns has equal norms, the tie of the rotation angle
    g = synth.lowrank_exp(512, 256, decay=0.0, noise_std=0.0, seed=l, K=l)
    Sd, _ = upload(g["St"], torch.float64)
    Phi, sig, A = run_gpu(Sd, 512, 256, l, 0, 1, 3, torch.float64)
    assert np.max(np.abs(sig - 1.0)) <= 1e-12
    assert np.max(np.abs(Phi.T @ Phi - np.eye(l))) <= 1e-12
    assert np.max(np.abs(Phi @ A - g["St"].T)) <= 1e-11
