"""Projections whose blocks are of one order class, each class with its own
launch shape, and of several classes in more blocks than the device has compute
units: against numpy in float64 with the tolerances of the edge tests, and
block by block the same eigenvalues as from the one-launch form (float64,
backward stable: 1e-12)."""
import numpy as np
import pytest
import torch

from gpu_common import ensure_lib, say
from test_gpu_eig_edges import _matrix

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
CLASSES = {"to 32": (1, 2, 7, 8, 9, 16, 17, 25, 31, 32), "to 64": (33, 47, 48, 49, 63, 64),
           "to 128": (65, 80, 81, 96, 97, 112, 113, 127, 128), "all, many": (1, 31, 32, 33, 64, 65) * 50}


@pytest.mark.parametrize("name", list(CLASSES))
@pytest.mark.parametrize("kind", ["random", "clusters"])
def test_classes(name, kind):
    ensure_lib()
    from paper_2606_13825_amd import psd_proj
    from synth import svec_of_dense
    rng, orders = np.random.default_rng(13), CLASSES[name]
    mats = [0.5 * (S + S.T) for S in (_matrix(rng, p, kind) for p in orders)]
    vs = [svec_of_dense(S) for S in mats]
    x = lambda idx: torch.from_numpy(np.concatenate([vs[i] for i in idx])).to(DEV)
    say(f"eigensolver classes: {name}, {kind}")
    every = list(range(len(orders)))
    out, lam, _ = psd_proj(x(every), list(orders))
    some = every[:6] + [every[-1]]   # with a block of another class: one launch
    extra = [40, 20] if orders[0] > 64 else [100, 80]
    ex = torch.from_numpy(np.concatenate([svec_of_dense(np.eye(p)) for p in extra])).to(DEV)
    _, lam1, _ = psd_proj(torch.cat([x(some), ex]), [orders[i] for i in some] + extra)
    out, lam, lam1 = (t.cpu().numpy() for t in (out, lam, lam1))
    ro = lo = 0
    first = []
    for p, S in zip(orders, mats):
        nr = p * (p + 1) // 2
        w, V = np.linalg.eigh(S)
        ref = svec_of_dense((V * np.maximum(w, 0)) @ V.T)
        scale = np.linalg.norm(S)
        assert np.linalg.norm(out[ro:ro + nr] - ref) <= 1e-12 * scale, (p, "projection")
        assert np.abs(np.sort(lam[lo:lo + p]) - w).max() <= 1e-12 * scale, (p, "eigenvalues")
        first.append(lo)
        ro, lo = ro + nr, lo + p
    lo = 0
    for i in some:
        p = orders[i]
        a, b = np.sort(lam[first[i]:first[i] + p]), np.sort(lam1[lo:lo + p])
        assert np.abs(a - b).max() <= 1e-12 * np.linalg.norm(mats[i]), (p, "one launch")
        lo += p
