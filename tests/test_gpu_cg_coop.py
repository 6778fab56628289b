"""The cooperative CG on plans that run it -- more instances than compute
units, and a vector too long for a workgroup's LDS -- against the float64
oracle.  Tolerances as for the teams: float64 solves stop at a relative residual
of 1e-12 and condition numbers are below 1e4, so 1e-8 for iterates and 1e-7 for
gradients; float32 the contract's 1e-5 and 1e-4."""
import numpy as np
import pytest
import torch

import synth
from gpu_common import assert_close, ensure_lib, floor_of, oracle_run, say
from test_host_cg_kernel import _sparse

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("name,dtype,tol_it,tol_g", [("device full", torch.float64, 1e-8, 1e-7),
                                                     ("device full", torch.float32, 1e-5, 1e-4),
                                                     ("long vector", torch.float64, 1e-8, 1e-7)])
def test_cooperative_cg_matches_oracle(name, dtype, tol_it, tol_g):
    ensure_lib()
    from paper_2606_13825_amd import CosmoBatch
    npdt = np.float64 if dtype == torch.float64 else np.float32
    rng = np.random.default_rng(19)
    insts = _sparse(rng, 40, 50, 6, B=300) if name == "device full" else _sparse(rng, 20500, 3000, 4)
    insts = [i.astype(npdt) for i in insts]
    hyper = [synth.perturbed_hyper(i, 2, rng) for i in insts]
    hyper = [(r.astype(npdt), np.asarray(a).astype(npdt)) for r, a in hyper]
    batch = CosmoBatch(insts, K=2, dtype=dtype, device=DEV, cg_tol=1e-12 if npdt is np.float64 else 1e-8)
    batch.set_pcg_form(4)
    assert batch.cg_kernel()[0] == "cooperative"
    say(f"cooperative CG: {name}, {dtype}")
    rho = torch.from_numpy(np.concatenate([h[0] for h in hyper], axis=1)).to(DEV)
    alpha = torch.from_numpy(np.stack([h[1] for h in hyper], axis=1)).to(DEV)
    stats = batch.new_stats()
    fw = batch.forward(rho, alpha, stats=stats)
    _, g = batch.residual_loss(fw.x, fw.s, fw.y)
    bw = batch.backward(rho, alpha, fw.tape, *g, stats=stats)
    torch.cuda.synchronize()
    assert batch.stats_dict(stats)["nonfinite"].sum() == 0
    for i in range(0, len(insts), 23):
        ref, fl = oracle_run(insts[i], *hyper[i]), floor_of(insts[i])
        n, m = slice(batch.n_off[i], batch.n_off[i + 1]), slice(batch.m_off[i], batch.m_off[i + 1])
        for nm, t, tol in (("x", fw.x[n], tol_it), ("s", fw.s[m], tol_it), ("y", fw.y[m], tol_it),
                           ("grho", bw.grho[:, m], tol_g), ("gx0", bw.gx0[n], tol_g), ("gs0", bw.gs0[m], tol_g),
                           ("gy0", bw.gy0[m], tol_g)):
            assert_close(t.cpu().numpy(), ref[nm], tol, fl, f"instance {i} {nm}")
