"""The Cholesky factorisation that follows the reduction of a Gram matrix, at every
padded width of the sketch (1 to 8 blocks of 16, whole and partial last blocks):
the shifted retry when the sketch is wider than the rank, and the count of finished
workgroups, which has to be back at zero after every launch (the second call). Plain
factorisations at every width are in the small SVD's tests. Against the exact POD, with the tolerances of the rank-deficient parity test."""

import numpy as np
import pytest
import torch

import paper_2504_15350_amd as rp
import synth
from oracle import metrics, pod
from test_gpu_parity import DEV, upload

pytestmark = pytest.mark.gpu


def _rank(m, n, k, seed):
    U, V = synth._orthonormal(m, k, seed, 1), synth._orthonormal(n, k, seed, 2)
    return (V * np.linspace(2.0, 1.0, k)) @ U.T


@pytest.mark.parametrize("l", [2, 16, 17, 32, 48, 63, 64, 65, 80, 96, 112, 127, 128])
def test_shifted_retry_at_every_width(l):
    k = max(1, l // 3)
    Sd, S64 = upload(_rank(1500, 300, k, l), torch.float64)
    plan = rp.Plan(1500, 300, k, l - k, 1, dtype=torch.float64, device=DEV)
    first = [t.clone() for t in plan.compute(Sd, 5)]
    flags = plan.status()
    again = [t.clone() for t in plan.compute(Sd, 5)]
    plan.close()
    print(f"[case] l={l} rank={k} flags={flags}", flush=True)
    # the trailing pivots are rounding errors of the Gram matrix (a few u), the limit is 2 l u
    assert l < 16 or flags & rp.FLAG_SHIFTED
    assert not flags & (rp.FLAG_BREAKDOWN | rp.FLAG_NONFINITE)
    assert all(torch.equal(a, b) for a, b in zip(first, again))
    P1, s1, _, _ = pod.pod_svd(S64, k)
    assert metrics.sigma_rel_err(first[1].cpu().numpy(), s1) < 1e-5
    assert metrics.sin_theta_max(first[0].cpu().numpy().T, P1) < 1e-4
