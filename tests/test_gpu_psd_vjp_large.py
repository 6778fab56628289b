"""The Daleckii-Krein VJP of blocks above order 128, at the edges of its tiles,
against the same formula in numpy float64 with the same eigenpairs.

Tolerances, relative to ||g||: four chained products of order p add errors of
about sqrt(p) eps each, 4 x 14 x 6e-8 = 3.4e-6 in float32 (1e-5 allowed) and
5e-15 in float64 (1e-13 allowed)."""
import numpy as np
import pytest
import torch

from gpu_common import ensure_lib, say

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("dtype,orders,tol", [
    (np.float32, (129, 130, 143, 144, 145, 159, 160, 161, 176, 177, 191, 192, 193, 197, 199, 200), 1e-5),
    (np.float64, (129, 131, 133, 136, 137, 139, 140), 1e-13),
])
def test_large_vjp(dtype, orders, tol):
    ensure_lib()
    from paper_2606_13825_amd import psd_proj_vjp
    from synth import svec_of_dense
    rng = np.random.default_rng(17)
    lams, Us, gs, refs = [], [], [], []
    for p in orders:
        U = np.linalg.qr(rng.standard_normal((p, p)))[0].astype(dtype)
        lam = rng.standard_normal(p).astype(dtype)
        lam[: p // 5], lam[p // 5: p // 4] = lam[0], 0.0
        G = rng.standard_normal((p, p))
        g = svec_of_dense(G + G.T).astype(dtype)
        u, l = U.astype(np.float64), lam.astype(np.float64)
        pos = l > 0
        den = np.abs(l)[:, None] + np.abs(l)[None, :]
        W = np.where(pos[:, None] & pos[None, :], 1.0, 0.0)
        mixed = pos[:, None] != pos[None, :]
        W[mixed] = (np.maximum(l[:, None], l[None, :]) / np.where(den > 0, den, 1.0))[mixed]
        S = np.zeros((p, p))
        iu = np.triu_indices(p)
        k = iu[1] * (iu[1] + 1) // 2 + iu[0]
        S[iu] = g.astype(np.float64)[k] * np.where(iu[0] == iu[1], 1.0, np.sqrt(0.5))
        S = S + np.triu(S, 1).T
        refs.append(svec_of_dense(u @ (W * (u.T @ S @ u)) @ u.T))
        lams.append(lam)
        Us.append(U.T.ravel())
        gs.append(g)
    say(f"large VJP {np.dtype(dtype).name}")
    t = lambda parts: torch.from_numpy(np.concatenate(parts)).to(DEV)
    out = psd_proj_vjp(t(lams), t(Us), t(gs), list(orders)).double().cpu().numpy()
    at = 0
    for p, g, ref in zip(orders, gs, refs):
        n = p * (p + 1) // 2
        assert np.linalg.norm(out[at:at + n] - ref) <= tol * np.linalg.norm(g), p
        at += n
