"""The FP64 leaf kernel's complex field (the transposed operator) with four,
two and one waves per leaf and leaves of few targets, against the oracle's
rows, and its time against the forward operator's where leaves are small.

Tolerance 1e-10 (max-norm relative): an expansion of 30 terms at the largest
separation ratio of the lists, about 0.47, leaves 0.47^30 ~ 1.5e-10 of a far
box's share of the field, and that share is well below one."""
import numpy as np
import pytest

import synth
from oracle import nystrom
from oracle.geometry import Curves

pytestmark = pytest.mark.gpu


def _stars(nodes):
    return synth.star_islands(71, 40, (0.04, 0.1), nodes=nodes)


# four waves a leaf below 2048 leaves, two below 8192, then one
@pytest.mark.parametrize("nodes,leaf,lo,hi", [(64, 4, 0, 1500), (200, 8, 1000, 2047),
                                              (300, 4, 2048, 8191), (700, 4, 8192, 20000)])
def test_field(nodes, leaf, lo, hi):
    import torch
    from paper_1306_0612_amd import lbs
    isl = _stars(nodes)
    cv = Curves(isl)
    sol = lbs.Solver(isl, leaf_max=leaf)
    assert lo <= sol.tree_info()["leaves"] <= hi
    rng = np.random.default_rng(72)
    rows = rng.choice(cv.n, size=min(cv.n, 200), replace=False)
    x = np.zeros(cv.n)
    x[rows] = rng.normal(size=len(rows))
    y = sol.matvec(torch.tensor(x, device="cuda"), "iplusk_t", "fp64").cpu().numpy()
    ref = x[rows] @ nystrom.kernel_block(cv, rows) + x
    assert np.abs(y - ref).max() < 1e-10 * np.abs(ref).max()
    sol.close()


def test_time_of_small_leaves():
    """8000 nodes in leaves of at most eight: the transposed application takes
    1.08 of the forward one's time; 1.25 when one lane adds all slices of a
    target."""
    import torch
    from paper_1306_0612_amd import lbs
    isl = _stars(200)
    sol = lbs.Solver(isl, leaf_max=8)
    x = torch.ones(sol.n_nodes, dtype=torch.float64, device="cuda")
    us = {}
    for op in ("iplusk", "iplusk_t", "iplusk", "iplusk_t", "iplusk", "iplusk_t"):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        for _ in range(50):
            sol.matvec(x, op, "fp64")
        b.record()
        b.synchronize()
        us[op] = min(us.get(op, 1e9), a.elapsed_time(b) * 20)
    assert us["iplusk_t"] < 1.17 * us["iplusk"], us
    sol.close()
