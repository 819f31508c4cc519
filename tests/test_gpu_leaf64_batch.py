"""FP64 applications of batches whose leaves have at most one stage of
sources (one wave per leaf) or a little more, forward and transposed, against
the oracle, and the time of the first sort.

Tolerance 1e-10 (max-norm relative): an expansion of 30 terms at the largest
separation ratio of the lists, about 0.47, leaves 0.47^30 ~ 1.5e-10 of a far
box's share of the field, and that share is well below one."""
import numpy as np
import pytest

import synth
from oracle import nystrom
from oracle.geometry import Curves

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("geoms,nodes", [(200, 64), (300, 64), (300, 128), (300, 129), (1100, 33)])
def test_values(geoms, nodes):
    import torch
    from paper_1306_0612_amd import lbs
    one = synth.cap_island(n=nodes)
    cv = Curves(one)
    A = nystrom.kernel_block(cv, np.arange(cv.n)) + np.eye(cv.n)
    sol = lbs.Solver([one] * geoms)
    X = np.random.default_rng(81).normal(size=(geoms, cv.n))
    x = torch.tensor(X.ravel(), device="cuda")
    for op, M in (("iplusk", A.T), ("iplusk_t", A)):
        y = sol.matvec(x, op, "fp64").cpu().numpy().reshape(geoms, cv.n)
        ref = X @ M
        assert (np.abs(y - ref).max(1) < 1e-10 * np.abs(ref).max(1)).all(), op
    sol.close()


def test_time():
    """2000 caps of 64 nodes: the transposed FP64 application takes 0.50 of
    the mixed one's time with one wave per leaf (38 and 77 us), 0.59 with
    two."""
    import torch
    from paper_1306_0612_amd import lbs
    sol = lbs.Solver([synth.cap_island(n=64)] * 2000)
    x = torch.ones(sol.n_nodes, dtype=torch.float64, device="cuda")
    us = {}
    for k in range(16):
        op, prec = ("iplusk_t", "fp64") if k % 2 else ("iplusk", "mixed")
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        for _ in range(100):
            sol.matvec(x, op, prec)
        b.record()
        b.synchronize()
        us[op] = min(us.get(op, 1e9), a.elapsed_time(b) * 10)
    assert us["iplusk_t"] < 0.545 * us["iplusk"], us
    sol.close()
