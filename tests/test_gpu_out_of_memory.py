"""Solves whose Krylov vectors do not fit the card (65535 columns of 6000
nodes, restart 120: 380 GB) are refused with LBS_ERR_OUT_OF_MEMORY."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def _handle(lbs):
    return lbs.Solver(synth.star_islands(71, 3, (0.1, 0.2), nodes=2000), restart=120, leaf_max=64)


def _refused(lbs, sol, big):
    with pytest.raises(lbs.LBSError) as e:
        sol.solve(big, tol=1e-10, precision="fp64")
    assert e.value.status == "LBS_ERR_OUT_OF_MEMORY"


def test_the_error_does_not_stay():
    """The failed allocation is this call's error alone, not also that of the
    program's next use of the GPU."""
    import torch
    from paper_1306_0612_amd import lbs
    sol = _handle(lbs)
    big = torch.zeros((65535, sol.n_nodes), dtype=torch.float64, device="cuda")
    _refused(lbs, sol, big)
    del big
    assert float((torch.ones(7, device="cuda") + 1).sum()) == 14.0
    sol.close()


def test_refused_again_and_usable_after():
    """The same call is refused again, and the handle then solves a smaller
    one as a new handle does."""
    import torch
    from paper_1306_0612_amd import lbs
    sol = _handle(lbs)
    big = torch.zeros((65535, sol.n_nodes), dtype=torch.float64, device="cuda")
    for _ in range(2):
        _refused(lbs, sol, big)
    del big
    g = torch.tensor(np.random.default_rng(72).normal(size=(2, sol.n_nodes)), device="cuda")
    s, a, _ = sol.solve(g, tol=1e-10, precision="fp64")
    sol.close()
    ref = _handle(lbs)
    s2, a2, _ = ref.solve(g, tol=1e-10, precision="fp64")
    assert torch.equal(s, s2) and torch.equal(a, a2)
    ref.close()
