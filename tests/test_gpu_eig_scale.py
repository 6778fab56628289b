"""Projections of very large and very small blocks.  A power of two times a
block has that power times its eigenvalues and projection and the same
eigenvectors, and every operation of the eigensolver scales exactly, so
results at any scale are bitwise those at scale one, as long as the sum of
squares of the entries stays in the data type's range (in float64, up to about
2^480 at these orders).  The result at scale one is compared with numpy in
float64: rotations leave an error of a few units in the last place per sweep,
well below 1e-13 ||S|| in float64; float32 outputs are rounded once, 1e-6."""
import numpy as np
import pytest
import torch

from gpu_common import ensure_lib, say

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
ORDERS = {np.float64: [1, 2, 20, 33, 60, 100, 128, 135, 140], np.float32: [1, 2, 20, 33, 60, 100, 128, 135, 200]}
# 10^12, 10^40, 10^60, 10^75, 10^144 and their inverses, nearly
POWERS = {np.float64: [40, 132, 200, 250, 480, -40, -132, -200, -250, -480], np.float32: [40, -40, -100]}


def _svec(S):
    j, i = np.tril_indices(S.shape[0])   # column by column, rows up to the diagonal
    return np.where(i == j, S[i, j], S[i, j] * np.sqrt(2.0))


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("together", [True, False], ids=["one call", "one call each"])
def test_projection_at_any_scale(dtype, together):
    ensure_lib()
    from paper_2606_13825_amd import binding as api
    rng = np.random.default_rng(12)
    mats = []
    for p in ORDERS[dtype]:
        G = rng.standard_normal((p, p))
        mats.append((G + G.T) / 2)
    vs = [_svec(M).astype(dtype) for M in mats]
    gs = [torch.from_numpy(rng.standard_normal(v.size).astype(dtype)).to(DEV) for v in vs]
    groups = [list(range(len(vs)))] if together else [[k] for k in range(len(vs))]

    def run(group, power):
        v = torch.from_numpy(np.ldexp(np.concatenate([vs[k] for k in group]), power)).to(DEV)
        orders = [ORDERS[dtype][k] for k in group]
        out, lam, U = api.psd_proj(v, orders)
        gin = api.psd_proj_vjp(lam, U, torch.cat([gs[k] for k in group]), orders)
        return [t.cpu().numpy() for t in (out, lam, U, gin)]

    for group in groups:
        say(f"projection at scales, {np.dtype(dtype).name}, orders {[ORDERS[dtype][k] for k in group]}")
        one = run(group, 0)
        at = 0
        for k in group:
            S = np.zeros_like(mats[k])
            j, i = np.tril_indices(S.shape[0])
            S[i, j] = S[j, i] = np.where(i == j, vs[k].astype(np.float64), vs[k].astype(np.float64) / np.sqrt(2.0))
            w, Q = np.linalg.eigh(S)
            want = _svec((Q * np.maximum(w, 0)) @ Q.T)
            err = np.linalg.norm(one[0][at:at + want.size] - want)
            assert err <= (1e-13 if dtype is np.float64 else 1e-6) * np.linalg.norm(S), (ORDERS[dtype][k], err)
            at += want.size
        for power in POWERS[dtype]:
            got = run(group, power)
            for nm, a, b, e in zip(("out", "eigenvalues", "eigenvectors", "cotangent"), got, one, (power, power, 0, 0)):
                assert np.array_equal(a, np.ldexp(b, e)), f"{nm} at 2^{power}, orders {[ORDERS[dtype][k] for k in group]}"
