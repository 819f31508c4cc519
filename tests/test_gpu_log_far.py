"""The system operator's log-source columns at island counts around the far
lists' chunks (64 entries) and a wave's step of four chunks, one and three
right-hand sides, against the oracle's kernel.

Tolerance: densities zero, so what is left is the expansion's tail (2.5e-16
of a term) and the rounding of M terms: (M + 60) 2^-52 of the sum of the
terms' sizes, at most 4e-14 of it here, held to 1e-13 of the largest value
of |A| sum |G|."""
import numpy as np
import pytest

import synth
from oracle.geometry import Curves
from oracle.nystrom import greens

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,rhs", [(1, 1), (2, 3), (64, 1), (66, 3), (130, 1), (256, 1), (258, 1),
                                   (322, 3)])
def test_island_counts(m, rhs):
    import torch
    from paper_1306_0612_amd import lbs
    isl = synth.star_islands(83, m, (0.01, 0.02), nodes=12, gap_factor=1.0)
    cv = Curves(isl)
    A = np.random.default_rng(84).normal(size=(rhs, m))
    x = np.concatenate([np.zeros((rhs, cv.n)), A], axis=1)
    sol = lbs.Solver(isl)
    y = sol.matvec(torch.tensor(x, device="cuda"), "system", "fp64").cpu().numpy()
    G = 2.0 * greens(cv.x, isl.center)
    size = (np.abs(G) @ np.abs(A).T).max(0)
    err = np.abs(y[:, :cv.n] - A @ G.T).max(1)
    assert (err < 1e-13 * size).all(), err / size
    sol.close()
