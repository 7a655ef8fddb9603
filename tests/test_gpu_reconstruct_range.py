"""FP32 reconstruction at the ends of FP32's range: infinities, NaN and values past
BF16's largest in the modes, the coefficients or the mean give what FP32 arithmetic
gives (an infinity stays one), and modes near or below the smallest normal number
lose no digits, on both entry points, with the coefficients split once or by every
workgroup, for rows on and off a multiple of four. Against the sums in FP64;
tolerance 2e-6 of the terms' magnitudes (the parity test's) and one unit of the
smallest number per term."""

import numpy as np
import pytest
import torch

import paper_2504_15350_amd as rp
from test_gpu_reconstruct import DEV

pytestmark = pytest.mark.gpu


def fields(Phi, alpha, mean, noalloc):
    (m, r), T = Phi.shape, alpha.shape[1]
    t = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to(DEV)
    args = t(Phi.T), t(alpha.T), t(mean) if mean is not None else None
    if not noalloc:
        return rp.reconstruct(*args)[0].cpu().numpy().T
    out = torch.empty((T, m), dtype=torch.float32, device=DEV)
    st = rp.lib().rpod_reconstruct_noalloc(rp._DTYPES[torch.float32], m, r, T, rp._dev_ptr(args[0]),
                                           rp._dev_ptr(args[2]) if mean is not None else None, rp._dev_ptr(args[1]),
                                           rp._dev_ptr(out), None, m, rp._stream_ptr(None, out.device)[0], None)
    torch.cuda.synchronize()
    assert st == 0
    return out.cpu().numpy().T


def check(F, Phi, alpha, mean):
    with np.errstate(all="ignore"):
        P, a = Phi.astype(np.float64), alpha.astype(np.float64)
        b = mean.astype(np.float64)[:, None] if mean is not None else np.zeros((Phi.shape[0], 1))
        ref = b + sum(P[:, k:k + 1] * a[k:k + 1] for k in range(P.shape[1]))
        mag = np.abs(b) + np.abs(P) @ np.abs(a)
    assert np.array_equal(np.isnan(F), np.isnan(ref))
    inf = np.isinf(ref)
    assert np.array_equal(np.isinf(F), inf) and np.array_equal(F[inf], ref[inf])
    ok = np.isfinite(ref)
    assert np.all(np.abs(F[ok] - ref[ok]) <= 2e-6 * mag[ok] + (P.shape[1] + 1) * 2.0 ** -149)


@pytest.mark.parametrize("noalloc", [False, True])
@pytest.mark.parametrize("m,r,T", [(5, 3, 7), (1025, 20, 40), (4096, 50, 33), (4097, 96, 20), (2050, 128, 20), (60001, 40, 300)])
def test_not_finite(m, r, T, noalloc):
    rng = np.random.default_rng(m + r)
    Phi, alpha, mean = (rng.standard_normal(s).astype(np.float32) for s in ((m, r), (r, T), (m,)))
    big = np.float32(3.3999e38)  # rounds to an infinity in BF16
    print(f"[case] m={m} r={r} T={T} noalloc={noalloc}", flush=True)
    for what, rows in ((Phi, True), (alpha, False), (mean, True)):
        for v in (np.inf, -np.inf, np.nan, big):
            x = [Phi, alpha, mean]
            y = what.copy()
            at = tuple(int(rng.integers(0, n)) for n in y.shape)
            y[at] = v
            if v is big:  # weights that keep the sum in range
                w = (alpha if rows else Phi) * np.float32(0.125)
                x = [Phi, w, mean] if rows else [w, alpha, mean]
            x = [y if z is what else z for z in x]
            check(fields(*x, noalloc), *x)
    alpha[0, 0] = 0.0
    Phi[m // 2, 0] = np.inf  # inf * 0
    check(fields(Phi, alpha, None, noalloc), Phi, alpha, None)


@pytest.mark.parametrize("noalloc", [False, True])
@pytest.mark.parametrize("m,r,T", [(1025, 20, 40), (4096, 50, 33), (60001, 40, 300)])
@pytest.mark.parametrize("e", [-95, -105, -112, -120, -128])
def test_small(m, r, T, e, noalloc):
    rng = np.random.default_rng(m + r - e)
    Phi, alpha = rng.standard_normal((m, r)).astype(np.float32), rng.standard_normal((r, T)).astype(np.float32)
    print(f"[case] m={m} r={r} T={T} 2^{e} noalloc={noalloc}", flush=True)
    s = np.float32(2.0) ** np.float32(e)
    check(fields(Phi * s, alpha, None, noalloc), Phi * s, alpha, None)
    check(fields(Phi, alpha * s, None, noalloc), Phi, alpha * s, None)
