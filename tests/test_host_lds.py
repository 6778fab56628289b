"""Every kernel has been allowed the dynamic LDS it is launched with, whichever
kernels of the same signature ran before it in the process, and on every device
(host code over a runtime without a GPU)."""
import numpy as np
import scipy.sparse as sp
import torch

import synth
from dense_layouts import instance
from host_runtime import load


def _sparse(rng, n, m, per_row):
    cols = np.concatenate([rng.choice(n, per_row, replace=False) for _ in range(m)])
    A = sp.csr_matrix((rng.standard_normal(m * per_row), cols, np.arange(0, m * per_row + 1, per_row)), shape=(m, n))
    return synth.ConicInstance(sp.identity(n, format="csr"), rng.standard_normal(n), A, rng.standard_normal(m),
                               [synth.Cone("nonneg", m)], {})


def _psd(rng, p):
    m = p * (p + 1) // 2
    return synth.ConicInstance(sp.identity(m, format="csr"), rng.standard_normal(m), sp.identity(m, format="csr") * -1.0,
                               rng.standard_normal(m), [synth.Cone("psd", p)], {})


def test_dynamic_lds_is_allowed(host_lib, monkeypatch):
    rt = load(None, monkeypatch, host_lib)
    from paper_2606_13825_amd import CosmoBatch
    from paper_2606_13825_amd import binding as api
    big = set()
    for device in (0, 1):
        rt.device(device)
        for dtype in (torch.float32, torch.float64):
            rng = np.random.default_rng(1)
            rt.reset()
            programs = [[_sparse(rng, 16000, 500, 40)], [instance(rng, 0, 9000, 16, 2000)], [instance(rng, 0, 2500, 700, 9000)],
                        [instance(rng, 0, 2500, 1000, 8000)], [instance(rng, 0, 30, 1000, 5)], [instance(rng, 0, 30, 20, 5)],
                        [_psd(rng, 60), _psd(rng, 120), _psd(rng, 140)]]
            for insts in programs:
                batch = CosmoBatch(insts, K=1, dtype=dtype, device="cpu", dense_f32=False)
                batch.forward(torch.ones(1, batch.m_tot, dtype=dtype), torch.ones(1, len(insts), dtype=dtype), tape=False)
            for orders in ([100], [30, 100], [135]):
                v = torch.zeros(sum(p * (p + 1) // 2 for p in orders), dtype=dtype)
                _, lam, U = api.psd_proj(v, orders)
                api.psd_proj_vjp(lam, U, v, orders)
            for l in rt.launches():
                if l.lds > 65536:
                    assert l.allowed >= l.lds, f"device {device}: {l.name} with {l.lds} bytes, allowed {l.allowed}"
                    big.add(l.name)
    # several kernels of one signature really asked for more than the default
    assert sum("k_pcg_team" in n for n in big) >= 4, big
    assert sum("k_psd_" in n for n in big) >= 6, big
