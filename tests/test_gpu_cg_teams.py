"""The CG with several workgroups per instance, against the float64 oracle:
row lengths of every class (none, short, middle, long), a general P, dense
blocks whose slices end inside a placement, uneven instances, and more
instances than a launch has teams.  Sizes are large enough for the plan to
choose teams (the largest instance takes tens of microseconds per operator
application in one workgroup).

Tolerances: the solves stop at a relative residual of 1e-12; the condition
numbers here are below 1e4, so iterates are within 1e-8 and gradients, which
solve once more on them, within 1e-7."""
import numpy as np
import pytest
import scipy.sparse as sp
import torch

import synth
from gpu_common import assert_close, ensure_lib, floor_of, oracle_run, say

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _program(rng, n, m, density, long_rows=0, empty_col=False, full_p=False):
    A = sp.random(m, n, density=density, format="lil", random_state=np.random.RandomState(int(rng.integers(1 << 30))),
                  data_rvs=rng.standard_normal)
    for r in range(long_rows):   # longer than a middle row
        A[r, :] = rng.standard_normal(n) / np.sqrt(n)
    A[m - 1, :] = 0.0            # a row of zeros
    if empty_col:
        A[:, n - 1] = 0.0
    A = A.tocsr()
    A.eliminate_zeros()
    if full_p:
        G = sp.random(n, n, density=2.0 / n, format="csr", random_state=np.random.RandomState(7))
        P = (G @ G.T + sp.identity(n)).tocsr()
    else:
        P = sp.diags(rng.uniform(0.5, 2.0, n)).tocsr()
    cones = [synth.Cone("zero", 3), synth.Cone("nonneg", m - 3 - 12), synth.Cone("soc", 5), synth.Cone("soc", 7)]
    return synth.ConicInstance(P, rng.standard_normal(n), A, rng.standard_normal(m), cones, {})


def _cases():
    rng = np.random.default_rng(5)
    yield "one sparse program, long rows, general P", [_program(rng, 1500, 900, 0.03, long_rows=3, full_p=True)]
    yield "uneven instances, an empty column", [_program(rng, n, n // 2 + 20, 0.05, empty_col=i == 1)
                                                for i, n in enumerate((1200, 331, 60, 800))]
    yield "dense designs", [synth.huber_socp(rng, n_obs=o, n_coef=c, n_soc=7).astype(np.float32)
                            for o, c in ((601, 97), (333, 130), (64, 20))]
    yield "more instances than teams", [
        _program(rng, 1300, 700, 0.05) if i in (17, 90) else _program(rng, 160 + 7 * (i % 11), 120 + i % 13, 0.12)
        for i in range(150)]


@pytest.mark.parametrize("case", range(4))
@pytest.mark.parametrize("form", [0, 4])
def test_cg_teams_match_oracle(case, form):
    ensure_lib()
    from paper_2606_13825_amd import CosmoBatch
    name, insts = list(_cases())[case]
    dense = "dense" in name
    if dense and form:
        pytest.skip("dense blocks run form 0 only")
    K, rng = 2, np.random.default_rng(9)
    hyper = [synth.perturbed_hyper(i, K, rng, eq_scale=10.0) for i in insts]
    batch = CosmoBatch(insts, K=K, dtype=torch.float64, device=DEV, dense_f32=dense)
    batch.set_pcg_form(form)
    rho = torch.from_numpy(np.concatenate([h[0] for h in hyper], axis=1)).to(DEV)
    alpha = torch.from_numpy(np.stack([h[1] for h in hyper], axis=1)).to(DEV)
    say(f"cg teams: {name}, form {form}")
    runs = []
    for _ in range(2):
        stats = batch.new_stats()
        fw = batch.forward(rho, alpha, stats=stats)
        loss, g = batch.residual_loss(fw.x, fw.s, fw.y)
        bw = batch.backward(rho, alpha, fw.tape, *g, stats=stats)
        torch.cuda.synchronize()
        runs.append((fw, loss, bw))
    st = batch.stats_dict(stats)
    assert st["cg_not_converged"].sum() == 0 and st["nonfinite"].sum() == 0
    for a, b in ((runs[0][0].x, runs[1][0].x), (runs[0][2].grho, runs[1][2].grho)):
        assert torch.equal(a, b), "two runs on the same inputs differ"
    fw, loss, bw = runs[0]
    for i in range(0, len(insts), 1 if len(insts) < 10 else 17):
        ref = oracle_run(insts[i], *hyper[i])
        fl = floor_of(insts[i])
        n, m = slice(batch.n_off[i], batch.n_off[i + 1]), slice(batch.m_off[i], batch.m_off[i + 1])
        for nm, t, tol in (("x", fw.x[n], 1e-8), ("s", fw.s[m], 1e-8), ("y", fw.y[m], 1e-8), ("grho", bw.grho[:, m], 1e-7),
                           ("gx0", bw.gx0[n], 1e-7), ("gs0", bw.gs0[m], 1e-7), ("gy0", bw.gy0[m], 1e-7)):
            assert_close(t.cpu().numpy(), ref[nm], tol, fl, f"{name}: instance {i} {nm}")
        assert_close(bw.galpha[:, i].cpu().numpy(), ref["galpha"], 1e-7, 0.0, f"{name}: instance {i} galpha")


def test_cg_teams_replayed_and_on_two_streams():
    """Graph replays, and two plans solving at the same time on two streams:
    every result is bitwise that of the plan alone."""
    ensure_lib()
    from paper_2606_13825_amd import CosmoBatch
    rng = np.random.default_rng(6)
    K, plans = 2, []
    for q in range(2):
        insts = [_program(rng, 900 + 100 * i, 500, 0.04) for i in range(3)]
        batch = CosmoBatch(insts, K=K, dtype=torch.float64, device=DEV)
        hyper = [synth.perturbed_hyper(i, K, rng, eq_scale=10.0) for i in insts]
        rho = torch.from_numpy(np.concatenate([h[0] for h in hyper], axis=1)).to(DEV)
        alpha = torch.from_numpy(np.stack([h[1] for h in hyper], axis=1)).to(DEV)
        ws = batch.new_fwd_ws()
        out = tuple(torch.empty(k, dtype=torch.float64, device=DEV) for k in (batch.n_tot, batch.m_tot, batch.m_tot))
        alone = batch.forward(rho, alpha, tape=False).x.clone()
        torch.cuda.synchronize()
        plans.append((batch, rho, alpha, ws, out, alone))
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    for graph in (False, True):
        for p in plans:
            p[0].set_graph(graph)
        for _ in range(3):
            for p, s in zip(plans, streams):
                with torch.cuda.stream(s):
                    for _ in range(3):
                        p[0].forward(p[1], p[2], tape=False, ws=p[3], out=p[4])
            torch.cuda.synchronize()
            for p in plans:
                assert torch.equal(p[4][0], p[5])
