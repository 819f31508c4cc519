"""The P2L sums by a launch of their own: with 129 columns even one
work-group per column is over the 128 that the upward pass takes along.
Every column equals its own application (which sums them beside the pass).

Tolerance 1e-13: the same sums in the same order up to the split between
launches, and 1e3 roundings of one column at most."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p64", [20, 30, 48])
def test_columns(p64):
    import torch
    from paper_1306_0612_amd import lbs
    isl = synth.star_islands(92, 12, (0.05, 0.15), nodes=[60 + 17 * k for k in range(12)])
    sol = lbs.Solver(isl, leaf_max=4, p64=p64)
    assert sol.tree_info()["x_pairs"] > 0
    X = torch.tensor(np.random.default_rng(93).normal(size=(129, sol.n_nodes)), device="cuda")
    Y = sol.matvec(X, "iplusk", "fp64")
    for r in (0, 64, 128):
        y = sol.matvec(X[r].contiguous(), "iplusk", "fp64")
        assert float((Y[r] - y).abs().max()) < 1e-13 * float(y.abs().max())
    sol.close()
