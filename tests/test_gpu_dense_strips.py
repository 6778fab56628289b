"""Column products of dense blocks in narrow strips (few blocks) and in wide
ones (at least a strip per compute unit), at the edges of both, against the
float64 oracle.  Tolerances as for the other float64 unrolls with solves to
1e-12: 1e-8 for iterates, 1e-7 for gradients."""
import numpy as np
import pytest
import torch

import synth
from gpu_common import assert_close, ensure_lib, floor_of, oracle_run, say

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
SIZES = ((40, 8), (70, 31), (71, 32), (90, 33), (150, 64), (151, 65), (300, 129))   # observations, coefficients


@pytest.mark.parametrize("dense_f32", [True, False])
@pytest.mark.parametrize("B", [7, 270])
def test_dense_strips(B, dense_f32):
    ensure_lib()
    from paper_2606_13825_amd import CosmoBatch
    rng = np.random.default_rng(31)
    insts = [synth.huber_socp(rng, n_obs=SIZES[i % 7][0] if i < 7 else 30, n_coef=SIZES[i % 7][1] if i < 7 else 12, n_soc=2)
             .astype(np.float32) for i in range(B)]
    hyper = [synth.perturbed_hyper(i, 1, rng, eq_scale=10.0) for i in insts]
    batch = CosmoBatch(insts, K=1, dtype=torch.float64, device=DEV, dense_f32=dense_f32)
    rho = torch.from_numpy(np.concatenate([h[0] for h in hyper], axis=1)).to(DEV)
    alpha = torch.from_numpy(np.stack([h[1] for h in hyper], axis=1)).to(DEV)
    say(f"dense strips: {B} blocks, float32 storage {dense_f32}")
    stats = batch.new_stats()
    fw = batch.forward(rho, alpha, stats=stats)
    loss, g = batch.residual_loss(fw.x, fw.s, fw.y)
    bw = batch.backward(rho, alpha, fw.tape, *g, stats=stats)
    torch.cuda.synchronize()
    st = batch.stats_dict(stats)
    assert st["cg_not_converged"].sum() == 0 and st["nonfinite"].sum() == 0
    for i in list(range(7)) + ([100, B - 1] if B > 7 else []):
        ref, fl = oracle_run(insts[i], *hyper[i]), floor_of(insts[i])
        n, m = slice(batch.n_off[i], batch.n_off[i + 1]), slice(batch.m_off[i], batch.m_off[i + 1])
        for nm, t, tol in (("x", fw.x[n], 1e-8), ("s", fw.s[m], 1e-8), ("y", fw.y[m], 1e-8), ("grho", bw.grho[:, m], 1e-7),
                           ("gx0", bw.gx0[n], 1e-7), ("gs0", bw.gs0[m], 1e-7), ("gy0", bw.gy0[m], 1e-7)):
            assert_close(t.cpu().numpy(), ref[nm], tol, fl, f"instance {i} {nm}")
