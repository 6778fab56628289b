"""Float64 blocks are rotated by float64 angles: the only pair of an order-2
block is orthogonal to 47 bits or more after its first rotation, so the second
sweep is the last (an angle of 24 bits leaves a coupling of 1e-8, and a third
sweep to find the 1e-16 that the second leaves)."""
import numpy as np
import pytest
import scipy.sparse as sp
import torch

import synth
from gpu_common import assert_close, ensure_lib, floor_of, oracle_run

pytestmark = pytest.mark.gpu


def test_order_two_blocks_end_with_the_second_sweep():
    ensure_lib()
    from paper_2606_13825_amd import CosmoBatch
    rng = np.random.default_rng(2)
    insts = [synth.ConicInstance(sp.identity(3, format="csr"), rng.standard_normal(3), sp.identity(3, format="csr") * -1.0,
                                 rng.standard_normal(3), [synth.Cone("psd", 2)], {}) for _ in range(200)]
    hyper = [synth.perturbed_hyper(i, 1, rng) for i in insts]
    batch = CosmoBatch(insts, K=1, dtype=torch.float64, device="cuda:0")
    stats = batch.new_stats()
    fw = batch.forward(torch.from_numpy(np.concatenate([h[0] for h in hyper], axis=1)).cuda(),
                       torch.from_numpy(np.stack([h[1] for h in hyper], axis=1)).cuda(), stats=stats)
    torch.cuda.synchronize()
    st = batch.stats_dict(stats)
    assert st["eig_not_converged"].sum() == 0
    assert st["eig_sweeps_max"].max() <= 2
    for i in (0, 77, 199):
        ref = oracle_run(insts[i], *hyper[i], with_grad=False)
        assert_close(fw.s[3 * i:3 * i + 3].cpu().numpy(), ref["s"], 1e-13, floor_of(insts[i]), f"instance {i}")
