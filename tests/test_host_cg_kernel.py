"""Which kernel runs the CG in each form, and what the autotuner makes of it
(host code over a runtime without a GPU): forms that would launch the same
kernel as form 0 are not timed against it, so timing noise cannot leave a form
that refuses graph mode."""
import numpy as np
import pytest
import scipy.sparse as sp
import torch

import synth
from dense_layouts import instance
from host_runtime import load


def _sparse(rng, n, m, per_row, B=1):
    out = []
    for _ in range(B):
        cols = np.concatenate([rng.choice(n, per_row, replace=False) for _ in range(m)])
        A = sp.csr_matrix((rng.standard_normal(m * per_row), cols, np.arange(0, m * per_row + 1, per_row)), shape=(m, n))
        out.append(synth.ConicInstance(sp.identity(n, format="csr"), rng.standard_normal(n), A, rng.standard_normal(m),
                                       [synth.Cone("nonneg", m)], {}))
    return out


def _plans():
    rng = np.random.default_rng(8)
    diag = synth.ConicInstance(sp.identity(9, format="csr"), rng.standard_normal(9), sp.identity(9, format="csr"),
                               rng.standard_normal(9), [synth.Cone("nonneg", 9)], {})
    # name: instances, kernel in form 0, kernel in the other forms (None: refused)
    yield "teams", _sparse(rng, 1500, 900, 40), "team", "team"
    yield "device full", _sparse(rng, 40, 50, 6, B=300), "workgroup", "cooperative"
    yield "vector too long for the LDS", _sparse(rng, 20500, 3000, 4), "workgroup", "cooperative"
    yield "more than 64 MB", _sparse(rng, 6000, 5500, 500), "team", "cooperative"
    yield "dense block", [instance(rng, 30, 8000, 12, 900)], "team", None
    yield "diagonal M", [diag], "none", "none"


NAMES = {"team": "k_pcg_team", "workgroup": "k_pcg", "cooperative": "k_pcg_coop", "none": None}


def _run(rt, batch, rho, alpha):
    rt.reset()
    batch.forward(rho, alpha, tape=False)
    used = {k for k, n in NAMES.items() if n and rt.launches(f"{len(n)}{n}I")}
    assert len(used) <= 1
    return used.pop() if used else "none"


@pytest.mark.parametrize("k", range(6))
def test_kernel_of_each_form_and_autotuner(host_lib, monkeypatch, k):
    rt = load(None, monkeypatch, host_lib)
    from paper_2606_13825_amd import CosmoBatch, CosmoError
    name, insts, form0, others = list(_plans())[k]
    batch = CosmoBatch(insts, K=1, dtype=torch.float64, device="cpu")
    rho, alpha = torch.ones(1, batch.m_tot, dtype=torch.float64), torch.ones(1, batch.B, dtype=torch.float64)
    for form in (0, 1, 2, 4):
        if form and others is None:
            with pytest.raises(CosmoError):
                batch.set_pcg_form(form)
            continue
        batch.set_pcg_form(form)
        want = others if form else form0
        assert batch.cg_kernel()[0] == want == _run(rt, batch, rho, alpha), (name, form)
    batch.set_pcg_form(0)
    assert (batch.cg_kernel()[1] > 1) == (form0 == "team")
    # the second and third schedules look faster than the first
    rt.elapsed([4.0, 1.0, 2.0, 3.0])
    form, ms = batch.autotune(rho, alpha)
    if others == "cooperative":
        assert form == 2 and ms[:4] == [4.0, 1.0, 2.0, 3.0]
    else:
        assert form == 0 and ms[1:3] == [-1.0, -1.0] and ms[0] == 4.0 and ms[3] == 1.0
        batch.set_graph(False)
        batch.set_graph(True)
    rt.elapsed([])
    batch.set_graph(False)
    if others:
        batch.set_pcg_form(1)   # explicit forms are accepted and refused as ever
        if others != "none":
            with pytest.raises(CosmoError, match="cooperative"):
                batch.set_graph(True)
