"""Programs with a narrow dense block among sparse columns, for the tests of
the team CG's dense columns."""
import numpy as np
import scipy.sparse as sp

import synth


def instance(rng, before, rows, cols, after, coupled=False):
    """`before` and `after` one-entry columns around a dense rows x cols block;
    coupled: every sparse column also meets a neighbour in a second row."""
    n, ns = before + cols + after, before + after
    G = sp.csr_matrix(rng.standard_normal((rows, cols)) / np.sqrt(rows))
    where = np.concatenate([np.arange(before), before + cols + np.arange(after)])
    S = sp.csr_matrix((rng.uniform(0.5, 1.5, ns), (np.arange(ns), where)), shape=(ns, n))
    parts = [S, sp.hstack([sp.csr_matrix((rows, before)), G, sp.csr_matrix((rows, after))])]
    if coupled and ns > 1:
        k = np.arange(ns - 1)
        parts.append(sp.csr_matrix((np.tile([0.6, -0.4], ns - 1), (np.repeat(k, 2), np.stack([where[:-1], where[1:]], 1).ravel())),
                                   shape=(ns - 1, n)))
        # and the block's first column meets a sparse one, so the parts are one system
        parts.append(sp.csr_matrix(([0.5, 0.5], ([0, 0], [where[0], before])), shape=(1, n)))
    A = sp.vstack(parts).tocsr()
    m = A.shape[0]
    P = sp.diags(rng.uniform(0.5, 2.0, n)).tocsr()
    inst = synth.ConicInstance(P, rng.standard_normal(n), A, rng.standard_normal(m), [synth.Cone("zero", 3), synth.Cone("nonneg", m - 3)],
                               {"dense": {"col0": before, "rows": rows, "cols": cols, "place": [(ns, 1.0)]}})
    inst.check()
    return inst
