"""FP32 matrices whose columns are too long for 32-bit byte offsets between them
(15 columns of 4 ld bytes pass 2^32 from ld = 71582789), with columns off the
128-byte lines. S has rank 16 and l = 16, so every column of the basis carries a
singular value. Against the singular value decomposition from the FP64 Gram
matrix S^T S (sigma_1 / sigma_16 = 4.5: no digits lost), with the FP32 tolerances
of the parity tests."""

import numpy as np
import pytest
import torch

import paper_2504_15350_amd as rp
from test_gpu_parity import DEV, TOL

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [72000003])
def test_columns_past_32_bit_offsets(m):
    n, l = 20, 16
    print(f"[case] m={m} n={n} l={l}", flush=True)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(5)
    V = np.linalg.qr(np.random.default_rng(5).standard_normal((n, l)))[0] * np.exp(-0.1 * np.arange(l))
    Vd = torch.from_numpy(V).to(DEV)
    St = torch.empty((n, m), dtype=torch.float32, device=DEV)
    step = 1 << 22
    blocks = [(i, min(i + step, m)) for i in range(0, m, step)]
    for i, j in blocks:
        St[:, i:j] = Vd.float() @ torch.randn((l, j - i), generator=gen, device=DEV)
    plan = rp.Plan(m, n, l, 0, 1, dtype=torch.float32, device=DEV)
    Phi, sig, A = plan.compute(St, 3)
    torch.cuda.synchronize()
    plan.close()
    G = torch.zeros((n, n), dtype=torch.float64, device=DEV)
    for i, j in blocks:
        B = St[:, i:j].double()
        G += B @ B.T.contiguous()
    w, W = np.linalg.eigh(G.cpu().numpy())
    s, W = np.sqrt(w[::-1][:l]), torch.from_numpy(np.ascontiguousarray(W[:, ::-1][:, :l])).to(DEV)
    U_scale = (W / torch.from_numpy(s).to(DEV)).T.contiguous()  # U^T = U_scale S^T
    PP, UP = (torch.zeros((l, l), dtype=torch.float64, device=DEV) for _ in range(2))
    for i, j in blocks:
        P, U = Phi[:, i:j].double(), U_scale @ St[:, i:j].double()
        PP += P @ P.T.contiguous()
        UP += U @ P.T.contiguous()
    tol = TOL[torch.float32]
    eye = torch.eye(l, dtype=torch.float64, device=DEV)
    assert np.max(np.abs(sig.cpu().numpy() - s) / s) <= tol["sigma"]
    assert float((PP - eye).abs().max()) <= tol["orth"]
    # every mode against its own: sin^2 = 1 - <u_k, phi_k>^2 for neighbours a gap of e^-0.1 apart
    cos = UP.diagonal().abs() / PP.diagonal().sqrt()
    assert float((1.0 - cos).max()) <= 0.5 * tol["sin"] ** 2 + 1e-12
    sgn = torch.sign(UP.diagonal())
    A_ref = sgn[:, None] * torch.from_numpy(s).to(DEV)[:, None] * W.T
    assert float((A.double().T - A_ref).norm() / A_ref.norm()) <= tol["A"]
