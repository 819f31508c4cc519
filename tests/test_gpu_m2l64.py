"""The FP64 M2L and P2L kernels over expansion orders and tree shapes (groups
of V-list entries, boxes with and without X lists, P2L beside the upward
pass and by a launch of its own) against the oracle's direct sums.

Tolerance: an expansion of p terms at the lists' largest separation ratio,
about 0.47, leaves 0.47^p of a far box's share of the field; rounding of the
sums adds 1e-13.  p = 20: 3e-7, 24: 1.4e-8, 30: 1.5e-10, 36: 1.6e-12, from 40
on the rounding."""
import numpy as np
import pytest

import synth
from oracle import nystrom
from oracle.geometry import Curves

pytestmark = pytest.mark.gpu

TOL = {20: 3e-7, 24: 1.4e-8, 30: 1.5e-10, 36: 1.7e-12, 40: 2e-13, 48: 2e-13}


def _rel(a, b):
    return np.abs(np.asarray(a) - np.asarray(b)).max() / np.abs(b).max()


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_1306_0612_amd import lbs
    lbs.load()
    return torch, lbs


def _geometry(name):
    if name == "tiny":    # hardly any V list
        return synth.star_islands(91, 2, (0.1, 0.2), nodes=[16, 9])
    return synth.star_islands(92, 12, (0.05, 0.15), nodes=[60 + 17 * k for k in range(12)])


@pytest.mark.parametrize("name,leaf", [("stars", 4), ("stars", 20), ("stars", 64), ("tiny", 4)])
@pytest.mark.parametrize("p64", sorted(TOL))
def test_orders_and_trees(env, name, leaf, p64):
    torch, lbs = env
    isl = _geometry(name)
    cv = Curves(isl)
    A = nystrom.kernel_block(cv, np.arange(cv.n)) + np.eye(cv.n)
    sol = lbs.Solver(isl, leaf_max=leaf, p64=p64)
    X = np.stack([synth.random_vector(s, cv.n) for s in (1, 2)])
    Y = sol.matvec(torch.tensor(X, device="cuda"), "iplusk", "fp64").cpu().numpy()
    assert _rel(Y, X @ A.T) < TOL[p64]
    Yt = sol.matvec(torch.tensor(X[0], device="cuda"), "iplusk_t", "fp64").cpu().numpy()
    assert _rel(Yt, X[0] @ A) < TOL[p64]


def test_p2l_by_its_own_launch(env):
    """Columns enough that the P2L sums leave the upward pass's launch; every
    column equal to its own application."""
    torch, lbs = env
    isl = _geometry("stars")
    sol = lbs.Solver(isl, leaf_max=4)
    assert sol.tree_info()["x_pairs"] > 0
    X = torch.tensor(np.stack([synth.random_vector(s, sol.n_nodes) for s in range(80)]),
                     device="cuda")
    Y = sol.matvec(X, "iplusk", "fp64").cpu().numpy()
    for r in (0, 41, 79):
        y = sol.matvec(X[r].contiguous(), "iplusk", "fp64").cpu().numpy()
        assert _rel(Y[r], y) < 1e-13
