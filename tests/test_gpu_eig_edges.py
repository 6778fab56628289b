"""The eigensolver at the edges of its launch shapes (column blocks, row
pieces, lane groups and order classes), against numpy in float64.

Tolerances.  float64: Jacobi is backward stable, p eps per sweep over about
ten sweeps at p <= 140 gives 1.6e-13 relative; 1e-12.  float32 up to order
128: the sweeps run in float64, so the projection is off by its rounding to
float32 (6e-8 of each entry) and U by 6e-8 of each entry (2.4e-7 in U'U
allows both factors and their sum).  float32 above 128: 2e-6, as
much as float32 sweeps with a refinement were allowed."""
import numpy as np
import pytest
import torch

from gpu_common import ensure_lib, say

pytestmark = pytest.mark.gpu

DEV = "cuda:0"

EDGES = (1, 2, 3, 4, 5, 7, 8, 9, 15, 16, 17, 23, 24, 25, 31, 32, 33, 47, 48, 49, 63, 64, 65, 72, 73, 79, 80, 81, 95, 96, 97,
         103, 104, 105, 111, 112, 113, 120, 121, 127, 128, 129, 136, 137, 139, 140)
LARGE = (129, 135, 144, 145, 160, 161, 176, 177, 192, 193, 199, 200)


def _matrix(rng, p, kind):
    if kind == "random":
        A = rng.standard_normal((p, p))
        return A + A.T
    if kind == "clusters":   # repeated eigenvalues of both signs
        Q = np.linalg.qr(rng.standard_normal((p, p)))[0]
        S = (Q * np.where(np.arange(p) % 2 == 0, 1.0, -1.0)) @ Q.T
        return S + S.T
    if kind == "zero":
        return np.zeros((p, p))
    if kind == "diagonal":
        return np.diag(rng.standard_normal(p))
    v = rng.standard_normal(p)   # rank one
    return np.outer(v, v)


@pytest.mark.parametrize("kind", ["random", "clusters", "zero", "diagonal", "rank1"])
@pytest.mark.parametrize("dtype,orders,tol,orth", [
    (np.float64, EDGES, 1e-12, 1e-12),
    (np.float32, [p for p in EDGES if p <= 128], 2e-7, 2.4e-7),
    (np.float32, LARGE, 2e-6, 2e-6),
])
def test_eigensolver_edges(dtype, orders, tol, orth, kind):
    ensure_lib()
    from paper_2606_13825_amd import psd_proj
    from synth import svec_of_dense
    rng = np.random.default_rng(11)
    mats, vs = [], []
    for p in orders:
        S = _matrix(rng, p, kind).astype(dtype).astype(np.float64)
        mats.append(0.5 * (S + S.T))
        vs.append(svec_of_dense(mats[-1]))
    say(f"eigensolver edges {np.dtype(dtype).name} {kind}")
    x = torch.from_numpy(np.concatenate(vs).astype(dtype)).to(DEV)
    out, lam, U = psd_proj(x, list(orders))
    torch.cuda.synchronize()
    out, lam, U, x = (t.double().cpu().numpy() for t in (out, lam, U, x))
    ro = uo = lo = 0
    for p, S in zip(orders, mats):
        nr = p * (p + 1) // 2
        w, V = np.linalg.eigh(S)
        ref = svec_of_dense((V * np.maximum(w, 0)) @ V.T)
        scale = max(np.linalg.norm(S), 1e-300)
        assert np.linalg.norm(out[ro:ro + nr] - ref) <= tol * scale, (p, "projection")
        assert np.abs(np.sort(lam[lo:lo + p]) - w).max() <= tol * scale, (p, "eigenvalues")
        Ub = U[uo:uo + p * p].reshape(p, p).T
        assert np.abs(Ub.T @ Ub - np.eye(p)).max() <= orth, (p, "orthogonality")
        ro, uo, lo = ro + nr, uo + p * p, lo + p


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_eigensolver_scale_range(dtype):
    """Blocks far from unit norm: the sweeps see them scaled to order one."""
    ensure_lib()
    from paper_2606_13825_amd import psd_proj
    from synth import svec_of_dense
    rng = np.random.default_rng(12)
    A = rng.standard_normal((40, 40))
    S = A + A.T
    for e in (-12, -6, 6, 12):
        Se = (S * 10.0 ** e).astype(dtype).astype(np.float64)
        v = svec_of_dense(Se)
        out, _, _ = psd_proj(torch.from_numpy(v.astype(dtype)).to(DEV), [40])
        w, V = np.linalg.eigh(Se)
        ref = svec_of_dense((V * np.maximum(w, 0)) @ V.T)
        assert np.linalg.norm(out.double().cpu().numpy() - ref) <= (1e-12 if dtype == np.float64 else 2e-7) * np.linalg.norm(v)
