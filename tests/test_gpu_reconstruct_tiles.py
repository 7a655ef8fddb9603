"""Reconstruction at the edges of its tiles: rows short of a vector, a wave and a
workgroup, modes around the matrix cores' K steps (the mean is one more for FP32),
times around the 16 and 32 of a step, and enough rows for the coefficients to be
split once (FP32). Against the oracle with the tolerances of the reconstruction's
parity test; the entry point without a workspace gives the same fields."""

import numpy as np
import pytest
import torch

import paper_2504_15350_amd as rp
from oracle.reconstruct import reconstruct, rel_l2_error_of_time_averages
from test_gpu_reconstruct import DEV

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("m,r,T,with_mean", [
    (1, 1, 1, True),
    (2, 3, 17, False),
    (3, 15, 16, True),
    (5, 16, 31, True),
    (127, 17, 32, False),
    (129, 31, 33, True),
    (255, 32, 15, True),
    (257, 33, 65, False),
    (511, 63, 64, True),
    (1025, 64, 9, True),
    (2051, 65, 70, True),
    (3000, 95, 40, False),
    (4097, 96, 48, True),
    (5003, 127, 33, True),
    (6401, 128, 100, True),
    (40002, 20, 300, True),
    (33001, 70, 520, True),
])
def test_tiles(m, r, T, with_mean, dtype):
    rng = np.random.default_rng(7 * m + r + T)
    npd = np.float64 if dtype == torch.float64 else np.float32
    Phi = rng.standard_normal((m, r)).astype(npd)
    alpha = rng.standard_normal((r, T)).astype(npd)
    mean = rng.standard_normal(m).astype(npd) if with_mean else None
    F_ref = reconstruct(Phi, alpha, mean)
    ref = (F_ref + 0.1 * rng.standard_normal((m, T))).astype(npd)
    t = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to(DEV)
    args = t(Phi.T), t(alpha.T), t(mean) if with_mean else None
    print(f"[case] m={m} r={r} T={T} mean={with_mean} {dtype}", flush=True)
    F_t, eps = rp.reconstruct(*args, t(ref.T))
    F = F_t.double().cpu().numpy().T
    tol = 1e-12 if dtype == torch.float64 else 2e-6
    assert np.max(np.abs(F - F_ref)) <= tol * np.max(np.abs(F_ref))
    e_ref = rel_l2_error_of_time_averages(ref, F_ref)
    assert abs(eps - e_ref) <= (1e-10 if dtype == torch.float64 else 1e-5) * e_ref
    out = torch.full((T, m), float("nan"), dtype=dtype, device=DEV)
    st = rp.lib().rpod_reconstruct_noalloc(rp._DTYPES[dtype], m, r, T, rp._dev_ptr(args[0]),
                                           rp._dev_ptr(args[2]) if with_mean else None,
                                           rp._dev_ptr(args[1]), rp._dev_ptr(out), None, m,
                                           rp._stream_ptr(None, out.device)[0], None)
    torch.cuda.synchronize()
    assert st == 0 and torch.equal(out, F_t)
