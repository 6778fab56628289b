"""A block's projection has the same bits whatever other blocks the call has:
alone, among its own class, or with blocks of other order classes (which share
one launch where they do not fill the device)."""
import numpy as np
import pytest
import torch

from gpu_common import ensure_lib, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_bits_do_not_depend_on_other_blocks(dtype):
    ensure_lib()
    from paper_2606_13825_amd import binding as api
    rng = np.random.default_rng(5)
    orders = [3, 17, 32, 33, 50, 64, 65, 100, 128, 135, 20, 20, 60, 90, 8, 31, 47]
    blocks = [torch.from_numpy(rng.standard_normal(p * (p + 1) // 2)).to("cuda:0", dtype) for p in orders]

    def split(v, sizes):
        return torch.split(v, sizes)

    def project(which):
        ps = [orders[k] for k in which]
        out, lam, U = api.psd_proj(torch.cat([blocks[k] for k in which]), ps)
        return list(zip(split(out, [p * (p + 1) // 2 for p in ps]), split(lam, ps), split(U, [p * p for p in ps])))
    say(f"bits of projections among others, {dtype}")
    together = project(range(len(orders)))
    n = len(orders)
    many = project([k % n for k in range(20 * n)])   # more blocks than compute units: class by class
    for k in range(n):
        alone = project([k])[0]
        for nm, a, b, c in zip(("out", "eigenvalues", "eigenvectors"), alone, together[k], many[k]):
            assert torch.equal(a, b), f"{nm} of block {k} (order {orders[k]}) among other classes"
            assert torch.equal(a, c), f"{nm} of block {k} (order {orders[k]}) in a call that fills the device"
