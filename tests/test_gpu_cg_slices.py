"""Slices of a team's CG at the edges of what a workgroup keeps in LDS: rows and
columns kept, rows only, neither; and columns whose rows are listed because
they lie far apart.  Against the float64 oracle, with the tolerances of the
other team tests (residuals of 1e-12, condition numbers below 1e4: 1e-8 for
iterates, 1e-7 for gradients, which solve once more on them)."""
import numpy as np
import pytest
import scipy.sparse as sp
import torch

import synth
from gpu_common import assert_close, ensure_lib, floor_of, oracle_run, say

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _random(rng, m, n, per_row):
    cols = np.concatenate([rng.choice(n, per_row, replace=False) for _ in range(m)])
    val = rng.standard_normal(m * per_row) / np.sqrt(per_row)
    return sp.csr_matrix((val, cols, np.arange(0, m * per_row + 1, per_row)), shape=(m, n))


def _staged(rng, m, n):
    """A band of short rows, and eight columns with an entry every fiftieth row."""
    i = np.repeat(np.arange(m), 6)
    j = np.minimum(i * (n - 8) // m + np.tile(np.arange(6), m), n - 9)
    A = sp.csr_matrix((rng.standard_normal(6 * m) / 2, (i, j)), shape=(m, n)).tolil()
    for c in range(8):
        A[c::50, n - 8 + c] = 1.0
    A = A.tocsr()
    A.sum_duplicates()
    return A


@pytest.mark.parametrize("name,m,n,per_row", [("rows and columns kept", 900, 1500, 40), ("rows kept", 1000, 1600, 320),
                                              ("nothing kept", 1100, 1800, 700), ("listed rows", 6000, 2400, 0)])
def test_cg_slices_match_oracle(name, m, n, per_row):
    ensure_lib()
    from paper_2606_13825_amd import CosmoBatch
    rng = np.random.default_rng(21)
    A = _random(rng, m, n, per_row) if per_row else _staged(rng, m, n)
    inst = synth.ConicInstance(sp.diags(rng.uniform(0.5, 2.0, n)).tocsr(), rng.standard_normal(n), A,
                               rng.standard_normal(m), [synth.Cone("zero", 3), synth.Cone("nonneg", m - 3)], {})
    rho, alpha = synth.perturbed_hyper(inst, 1, rng, eq_scale=10.0)
    batch = CosmoBatch([inst], K=1, dtype=torch.float64, device=DEV, dense=False)
    say(f"cg slices: {name}")
    stats = batch.new_stats()
    r, a = torch.from_numpy(rho).to(DEV), torch.from_numpy(np.atleast_1d(alpha).reshape(1, 1)).to(DEV)
    fw = batch.forward(r, a, stats=stats)
    loss, g = batch.residual_loss(fw.x, fw.s, fw.y)
    bw = batch.backward(r, a, fw.tape, *g, stats=stats)
    torch.cuda.synchronize()
    st = batch.stats_dict(stats)
    assert st["cg_not_converged"].sum() == 0 and st["nonfinite"].sum() == 0
    ref, fl = oracle_run(inst, rho, alpha), floor_of(inst)
    for nm, t, tol in (("x", fw.x, 1e-8), ("s", fw.s, 1e-8), ("y", fw.y, 1e-8), ("grho", bw.grho, 1e-7),
                       ("gx0", bw.gx0, 1e-7), ("gs0", bw.gs0, 1e-7), ("gy0", bw.gy0, 1e-7)):
        assert_close(t.cpu().numpy(), ref[nm], tol, fl, f"{name}: {nm}")
