"""The tables of the team CG, on the host.  For dense blocks that stand among
sparse columns: what a workgroup stores per dense column of its slice lies in
the region its LDS has for that.  For the rows that a slice's columns use: the
16-bit indices name those rows, in ranges, in lists and where a slice does not
fit; and every row is listed once."""
import numpy as np
import pytest
import torch

import scipy.sparse as sp

import synth
from dense_layouts import instance
from host_runtime import array, load

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


def _program(rng, m, n, per_row, far=0):
    """Random rows, or (far) a band and `far` columns with an entry every fiftieth row; some empty columns."""
    if far:
        i = np.repeat(np.arange(m), 6)
        j = np.minimum(i * (n - far) // m + np.tile(np.arange(6), m), n - far - 1)
        A = sp.coo_matrix((rng.standard_normal(6 * m), (i, j)), shape=(m, n)).tolil()
        for c in range(far):
            A[c::50, n - far + c] = 1.0
        A = A.tocsr()
    else:
        cols = np.concatenate([rng.choice(n - 7, per_row, replace=False) for _ in range(m)])
        A = sp.csr_matrix((rng.standard_normal(m * per_row), cols, np.arange(0, m * per_row + 1, per_row)), shape=(m, n))
    return synth.ConicInstance(sp.identity(n, format="csr"), rng.standard_normal(n), A, rng.standard_normal(m),
                               [synth.Cone("nonneg", m)], {})


PROGRAMS = {   # (m, n, entries per row, far columns) per instance
    "ranges": [(900, 1500, 40, 0)],
    "lists": [(6000, 2400, 0, 8), (5000, 1900, 0, 3)],
    "wide rows": [(1100, 1800, 700, 0), (300, 900, 300, 0)],
    "a slice that does not fit": [(60000, 9000, 40, 0)],
    "lists that do not fit": [(250000, 9000, 5, 0)],
    "uneven": [(800, 500, 25, 0), (17, 9, 2, 0), (2500, 1200, 30, 0)],
}


@pytest.mark.parametrize("dtype", [F64, F32])
@pytest.mark.parametrize("name", PROGRAMS)
def test_rows_of_slices(host_lib, monkeypatch, name, dtype):
    rt = load(None, monkeypatch, host_lib)
    from paper_2606_13825_amd import CosmoBatch
    rng = np.random.default_rng(6)
    tdt = torch.float32 if dtype is F32 else torch.float64
    insts = [_program(rng, *s).astype(dtype) for s in PROGRAMS[name]]
    batch = CosmoBatch(insts, K=1, dtype=tdt, device="cpu")
    rt.reset()
    batch.forward(torch.ones(1, batch.m_tot, dtype=tdt), torch.ones(1, batch.B, dtype=tdt), tape=False)
    t = rt.team(rt.launches("k_pcg_team")[0])
    kinds = set()
    for q in range(t["B"] * t["slices"]):
        ka, ke = t["At_rowptr"][t["colcut"][q]], t["At_rowptr"][t["colcut"][q + 1]]
        rows, loc = t["At_col"][ka:ke], t["At_loc"][ka:ke].astype(np.int64)
        first, cnt = int(t["used"][2 * q]), int(t["used"][2 * q + 1])
        distinct = np.unique(rows)
        if cnt * np.dtype(dtype).itemsize > t["cap"]:
            kinds.add("neither")
            assert cnt >= len(distinct)
        elif first < 0:
            kinds.add("list")
            assert cnt == len(distinct)
            listed = array(t["uses"] + 4 * (-1 - first), cnt, np.int32)
            np.testing.assert_array_equal(listed, distinct)
            np.testing.assert_array_equal(listed[loc], rows)
        elif cnt:
            kinds.add("range")
            assert first == distinct[0] and first + cnt == distinct[-1] + 1
            np.testing.assert_array_equal(first + loc, rows)
        else:
            assert ka == ke
    want = {"ranges": {"range"}, "lists": {"range", "list"}, "wide rows": {"range"}, "uneven": {"range"},
            "a slice that does not fit": {"neither"}, "lists that do not fit": {"neither"}}[name]
    assert want <= kinds, kinds
    assert sorted(t["rowsA"]) == list(range(t["m"]))
    BV = t["B"] * t["slices"]
    assert (np.diff(t["sliceA"]) >= 0).all() and t["sliceA"][0] == 0 and t["sliceA"][-1] == t["m"]
    assert all(t["sliceA"][c * (BV + 1)] == t["sliceA"][c * (BV + 1) - 1] for c in (1, 2))
