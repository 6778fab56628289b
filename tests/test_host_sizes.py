"""The sizes of standalone projections: the short way from a list to an int32
array gives what numpy gives, and leaves to numpy whatever it cannot read."""
import numpy as np
import pytest

from paper_2606_13825_amd import binding as api

SAME = [[], [1], [5] * 1000, [0, 255], [255, 256], [3, -1], [True, 2], (3, 4, 5), [np.int64(7), 8], [2.0, 3.9],
        [[1, 2], [3, 4]], np.array([4, 5], np.int64), np.array([4, 300], np.uint16), range(3, 9), [2 ** 31 - 1],
        ["7", "8"], b"", np.int32(4), 6, [np.array([3])], [np.array(3), 4]]


@pytest.mark.parametrize("sizes", SAME, ids=[repr(s)[:24] for s in SAME])
def test_same_as_numpy(sizes):
    try:
        want = np.asarray(sizes, np.int32)
    except Exception as e:
        with pytest.raises(type(e)):
            api._host_sizes(sizes)
        return
    got = api._host_sizes(sizes)
    assert got.dtype == np.int32 and got.shape == want.shape and got.flags.c_contiguous
    np.testing.assert_array_equal(got, want)


@pytest.mark.parametrize("bad", [[2 ** 31], [None], [1, "x"], [1 << 70], [[1], [2, 3]]])
def test_refused_as_numpy_refuses(bad):
    with pytest.raises(Exception) as want:
        np.asarray(bad, np.int32)
    with pytest.raises(want.type):
        api._host_sizes(bad)


def test_offsets_follow_the_orders():
    p = np.array([1, 2, 200, 46340, 7], np.int32)
    want = np.concatenate([[0], np.cumsum([int(q) * (int(q) + 1) // 2 for q in p])[:-1]])
    np.testing.assert_array_equal(api._packed_offsets(api._psd_rows(p.astype(np.int64))), want)
