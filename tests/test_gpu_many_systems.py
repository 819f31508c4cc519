"""Solves of batches with thousands of systems (many work-groups count them,
most Gram-Schmidt chunks hold a few rows) that converge after different
numbers of iterations, against the oracle's dense solves.

Tolerance: GMRES stops at a relative residual of 1e-12; the error in the
2-norm is at most the condition number (1.8e3 for the worst of the matrices
here) times that, and relative to the largest entry at most sqrt(100) = 10
times more: 2e-8."""
import numpy as np
import pytest

import synth
from oracle import nystrom
from oracle.geometry import Curves

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("geoms,cols", [(3, 1), (5, 1), (600, 3), (1501, 1)])
def test_batch(geoms, cols):
    import torch
    from paper_1306_0612_amd import lbs
    kinds = [synth.cap_island(n=16), synth.star_islands(75, 2, (0.1, 0.2), nodes=[33, 40]),
             synth.star_islands(76, 3, (0.1, 0.2), nodes=[24, 33, 40])]
    cvs = [Curves(s) for s in kinds]
    mats = [nystrom.system_matrix(c) for c in cvs]
    pick = np.random.default_rng(77).integers(3, size=geoms)
    n = sum(cvs[k].n for k in pick)
    G = np.random.default_rng(78).normal(size=(cols, n))
    sol = lbs.Solver([kinds[k] for k in pick])
    for prec in ("fp64", "mixed"):
        s, a, info = sol.solve(torch.tensor(G, device="cuda"), tol=1e-12, precision=prec)
        s, a = s.cpu().numpy(), a.cpu().numpy()
        no, io = sol.node_offsets, sol.island_offsets
        for q, k in enumerate(pick):
            rhs = np.concatenate([2 * G[:, no[q]:no[q + 1]], np.zeros((cols, cvs[k].m))], 1)
            ref = np.linalg.solve(mats[k], rhs.T).T
            got = np.concatenate([s[:, no[q]:no[q + 1]], a[:, io[q]:io[q + 1]]], 1)
            err = np.abs(got - ref).max(1) / np.abs(ref).max(1)
            assert (err < 2e-8).all(), (prec, q, k, err)
    sol.close()
