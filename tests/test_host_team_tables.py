"""The tables of the team CG for dense blocks that stand among sparse columns,
on the host: what a workgroup stores per dense column of its slice lies in the
region its LDS has for that."""
import numpy as np
import pytest
import torch

from dense_layouts import instance
from host_runtime import load

F32, F64 = np.float32, np.float64
LAYOUTS = [   # instances, dtype, (sparse columns before, rows, columns, sparse columns after)
    (32, F32, (6000, 3000, 16, 0)),
    (1, F32, (12000, 20000, 8, 0)),
    (1, F64, (3000, 8000, 8, 0)),
    (1, F64, (0, 8000, 8, 3000)),
    (2, F64, (1500, 6000, 12, 1700)),
    (3, F64, (5, 2000, 500, 0)),
]


@pytest.mark.parametrize("B,dtype,shape", LAYOUTS, ids=[f"{b}x{np.dtype(d).name}-{s}" for b, d, s in LAYOUTS])
def test_dense_columns_stay_in_their_region(host_lib, monkeypatch, B, dtype, shape):
    rt = load(None, monkeypatch, host_lib)
    from paper_2606_13825_amd import CosmoBatch
    rng = np.random.default_rng(3)
    tdt = torch.float32 if dtype is F32 else torch.float64
    batch = CosmoBatch([instance(rng, *shape).astype(dtype) for _ in range(B)], K=1, dtype=tdt, device="cpu")
    rt.reset()
    batch.forward(torch.ones(1, batch.m_tot, dtype=tdt), torch.ones(1, B, dtype=tdt), tape=False)
    launch, = rt.launches("k_pcg_team")
    t = rt.team(launch)
    assert launch.lds == t["cap_off"] + t["cap"]
    # the region behind the instance's vector (and before the kept slice)
    room = (t["cap_off"] - (t["max_n"] * np.dtype(dtype).itemsize + 7) // 8 * 8) // 8
    assert t["dense_slots"] <= room
    for q in range(B * t["slices"]):
        cols = np.arange(t["colcut"][q], t["colcut"][q + 1])
        dense = cols[t["dcol"][cols] >= 0]
        assert len(dense) <= t["dense_slots"]
        np.testing.assert_array_equal(t["dense_list"][t["dense_cut"][q]:t["dense_cut"][q + 1]], t["dcol"][dense])
        np.testing.assert_array_equal(t["dense_slot"][dense], np.arange(len(dense)))
        assert (t["dense_slot"][np.setdiff1d(cols, dense)] == -1).all()
    assert t["dense_cut"][-1] == B * shape[2]
