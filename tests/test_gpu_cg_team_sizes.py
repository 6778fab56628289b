"""Teams of every size give the same bits, and a team that gives up leaves no
instance that looks solved."""
import numpy as np
import pytest
import torch

import synth
from dense_layouts import instance
from gpu_common import ensure_lib, say
from test_gpu_cg_slices import _random, _staged
from test_gpu_cg_teams import _program

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _plain(rng, A):
    m, n = A.shape
    import scipy.sparse as sp
    return synth.ConicInstance(sp.diags(rng.uniform(0.5, 2.0, n)).tocsr(), rng.standard_normal(n), A, rng.standard_normal(m),
                               [synth.Cone("zero", 3), synth.Cone("nonneg", m - 3)], {})


def _insts(name):
    rng = np.random.default_rng(40)
    if name == "kept and listed rows":
        return [_plain(rng, _random(rng, 900, 1500, 40)), _plain(rng, _staged(rng, 6000, 2400)), _program(rng, 800, 500, 0.05, full_p=True)]
    if name == "nothing kept":
        return [_plain(rng, _random(rng, 1100, 1800, 700)), _plain(rng, _random(rng, 700, 1500, 320))]
    if name == "dense blocks":
        return [instance(rng, 300, 6000, 12, 900, coupled=True), instance(rng, 0, 3000, 90, 40, coupled=True)]
    return [_program(rng, 1300, 700, 0.05) if i % 20 == 3 else _program(rng, 160 + 7 * (i % 11), 120 + i % 13, 0.12)
            for i in range(60)]


NAMES = ["kept and listed rows", "nothing kept", "dense blocks", "more instances than teams"]


def _batch(name, dtype):
    from paper_2606_13825_amd import CosmoBatch
    npdt = np.float64 if dtype == torch.float64 else np.float32
    insts = [i.astype(npdt) for i in _insts(name)]
    rng = np.random.default_rng(41)
    hyper = [synth.perturbed_hyper(i, 1, rng, eq_scale=10.0) for i in insts]
    batch = CosmoBatch(insts, K=1, dtype=dtype, device=DEV)
    rho = torch.from_numpy(np.concatenate([h[0] for h in hyper], axis=1)).to(DEV, dtype)
    alpha = torch.from_numpy(np.stack([h[1] for h in hyper], axis=1)).to(DEV, dtype)
    z = [torch.full((k,), 0.25, dtype=dtype, device=DEV) for k in (batch.n_tot, batch.m_tot, batch.m_tot)]

    tape = batch.forward(rho, alpha, *z).tape   # every backward is that of a complete forward

    def run():
        stats = batch.new_stats()
        fw = batch.forward(rho, alpha, *z, stats=stats)
        bw = batch.backward(rho, alpha, tape, torch.ones_like(fw.x), torch.ones_like(fw.s), torch.ones_like(fw.y), stats=stats)
        torch.cuda.synchronize()
        return [t.cpu().numpy() for t in (fw.x, fw.s, fw.y, bw.grho, bw.gx0)], batch.stats_dict(stats)
    return batch, run


@pytest.mark.parametrize("name", NAMES)
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_results_do_not_depend_on_team_sizes(name, dtype):
    ensure_lib()
    batch, run = _batch(name, dtype)
    want, st = run()
    assert all(np.isfinite(w).all() for w in want)
    for members in (1, 2, 3, 7, 16, 31, 0):
        say(f"{name}, {dtype}: teams of {members}")
        batch.set_cg_team(members)
        got, st2 = run()
        for nm, a, b in zip(("x", "s", "y", "grho", "gx0"), got, want):
            assert np.array_equal(a, b), f"{nm} with teams of {members}"
        assert (st2["cg_iters_total"] == st["cg_iters_total"]).all()


@pytest.mark.parametrize("name", NAMES)
def test_instances_given_up_are_marked(name):
    """Members that wait for 10 ns give up, the more so the larger the team:
    every instance is then either solved, with the usual bits, or non-finite and
    counted; and the next solve is as if nothing had happened."""
    ensure_lib()
    batch, run = _batch(name, torch.float64)
    want, st = run()
    assert st["cg_not_converged"].sum() == 0
    lost = 0
    for members in (2, 8, 0):
        say(f"{name}: teams of {members} that give up")
        batch.set_cg_team(members, 10)
        got, st2 = run()
        for i in range(batch.B):
            n = slice(batch.n_off[i], batch.n_off[i + 1])
            for k, nm in ((0, "x"), (4, "gx0")):
                if not np.array_equal(got[k][n], want[k][n]):
                    assert np.isnan(got[k][n]).all(), f"instance {i}: {nm} neither solved nor marked"
                    assert st2["cg_not_converged"][i] >= 1
                    lost += 1
        batch.set_cg_team(members)
        got, st2 = run()
        assert st2["cg_not_converged"].sum() == 0
        for a, b in zip(got, want):
            assert np.array_equal(a, b)
    assert lost > 0
    batch.set_cg_team(1, 10)   # nobody to wait for
    got, st2 = run()
    assert st2["cg_not_converged"].sum() == 0 and np.array_equal(got[0], want[0])
