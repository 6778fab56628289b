"""Team CG with a narrow dense block behind, in front of and among sparse
columns, against the float64 oracle: the slices that hold the dense columns
then hold many others too.

Tolerances: float64 solves stop at a relative residual of 1e-12; the condition
numbers here are below 1e4, so iterates are within 1e-8 and gradients, which
solve once more on them, within 1e-7.  float32: the contract's 1e-5 and 1e-4."""
import numpy as np
import pytest
import torch

import synth
from dense_layouts import instance
from gpu_common import assert_close, ensure_lib, floor_of, oracle_run, say

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# (sparse columns before, rows, columns, sparse columns after) per instance, dtype, float32 blocks
CASES = {
    "last": ([(3000, 8000, 8, 0)], np.float64, False),
    "first": ([(0, 8000, 8, 3000)], np.float64, False),
    "middle, uneven": ([(1500, 6000, 12, 1700), (40, 900, 5, 700), (2100, 3000, 30, 1)], np.float64, True),
    "last, float32": ([(2500, 9000, 16, 0), (900, 7000, 8, 0)], np.float32, False),
}


@pytest.mark.parametrize("name", CASES)
def test_dense_columns_among_sparse_ones(name):
    ensure_lib()
    from paper_2606_13825_amd import CosmoBatch
    shapes, dtype, dense_f32 = CASES[name]
    rng = np.random.default_rng(17)
    insts = [instance(rng, *s, coupled=True).astype(np.float32 if dense_f32 else dtype) for s in shapes]
    hyper = [synth.perturbed_hyper(i, 1, rng, eq_scale=10.0) for i in insts]
    if dtype is np.float32:
        hyper = [(r.astype(dtype), np.asarray(a).astype(dtype)) for r, a in hyper]
    tdt = torch.float64 if dtype is np.float64 else torch.float32
    batch = CosmoBatch(insts, K=1, dtype=tdt, device=DEV, dense_f32=dense_f32, cg_max_iter=2000,
                       cg_tol=1e-12 if dtype is np.float64 else 1e-10)
    say(f"dense block {name}")
    rho = torch.from_numpy(np.concatenate([h[0] for h in hyper], axis=1)).to(DEV, tdt)
    alpha = torch.from_numpy(np.stack([h[1] for h in hyper], axis=1)).to(DEV, tdt)
    fw = batch.forward(rho, alpha)
    _, g = batch.residual_loss(fw.x, fw.s, fw.y)
    bw = batch.backward(rho, alpha, fw.tape, *g)
    torch.cuda.synchronize()
    it, gr = (1e-8, 1e-7) if dtype is np.float64 else (1e-5, 1e-4)
    for i, inst in enumerate(insts):
        ref, fl = oracle_run(inst, *hyper[i]), floor_of(inst)
        n, m = slice(batch.n_off[i], batch.n_off[i + 1]), slice(batch.m_off[i], batch.m_off[i + 1])
        for nm, t, tol in (("x", fw.x[n], it), ("s", fw.s[m], it), ("y", fw.y[m], it), ("grho", bw.grho[:, m], gr),
                           ("gx0", bw.gx0[n], gr), ("gs0", bw.gs0[m], gr), ("gy0", bw.gy0[m], gr)):
            assert_close(t.cpu().numpy(), ref[nm], tol, fl, f"{name}: instance {i} {nm}")
