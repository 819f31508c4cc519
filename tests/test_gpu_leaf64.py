"""The FP64 leaf kernel over its launch shapes (waves per leaf, right-hand
sides per work-group, targets per lane) against the oracle's direct sums.

Tolerance 1e-10 (max-norm relative): an expansion of 30 terms at the
largest separation ratio of the lists, about 0.47, leaves 0.47^30 ~ 1.5e-10
of a far box's share of the field, and that share is well below one."""
import numpy as np
import pytest

import synth
from oracle import nystrom
from oracle.geometry import Curves

pytestmark = pytest.mark.gpu


def _rel(a, b):
    return np.abs(np.asarray(a) - np.asarray(b)).max() / np.abs(b).max()


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_1306_0612_amd import lbs
    lbs.load()
    return torch, lbs


@pytest.fixture(scope="module")
def geometry():
    isl = synth.star_islands(71, 8, (0.08, 0.2), nodes=[257, 320, 33, 401, 288, 300, 350, 299])
    cv = Curves(isl)
    return isl, nystrom.kernel_block(cv, np.arange(cv.n)) + np.eye(cv.n)


# leaf sizes: 4 (tiny leaves), 8, 9, 16, 17, 32, 33, 64, 65 (two passes of
# targets), 300; columns 1 and 3
@pytest.mark.parametrize("leaf", [4, 8, 9, 16, 17, 32, 33, 64, 65, 300])
def test_field_over_leaf_sizes(env, geometry, leaf):
    torch, lbs = env
    isl, A = geometry
    sol = lbs.Solver(isl, leaf_max=leaf)
    X = np.stack([synth.random_vector(s, A.shape[0]) for s in (1, 2, 3)])
    xd = torch.tensor(X, device="cuda")
    for cols in (1, 3):
        Y = sol.matvec(xd[:cols].contiguous(), "iplusk", "fp64").cpu().numpy()
        assert _rel(Y, X[:cols] @ A.T) < 1e-10
    Yt = sol.matvec(xd[0].contiguous(), "iplusk_t", "fp64").cpu().numpy()
    assert _rel(Yt, X[0] @ A) < 1e-10


# about 900 leaves of at most 4 nodes: with a group per leaf and column 2,
# 12 and 26 columns run four, two and one wave each; 37 and 77 share groups
# of four columns (two waves, one wave; the last group partly filled)
@pytest.mark.parametrize("cols", [2, 12, 26, 37, 77])
def test_field_over_columns(env, geometry, cols):
    torch, lbs = env
    isl, A = geometry
    sol = lbs.Solver(isl, leaf_max=4)
    assert 830 < sol.tree_info()["leaves"] < 1000
    X = np.stack([synth.random_vector(s, A.shape[0]) for s in range(cols)])
    Y = sol.matvec(torch.tensor(X, device="cuda"), "iplusk", "fp64").cpu().numpy()
    assert _rel(Y, X @ A.T) < 1e-10
