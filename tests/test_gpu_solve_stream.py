"""Calls on a stream of their own while the device's null stream is busy:
what they clear is cleared on their own stream, in order with its use (a
clear on the null stream could come after it)."""
import time

import numpy as np
import pytest

import synth
from oracle import nystrom
from oracle.geometry import Curves

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def spin():
    """Cycles of the spinning kernel (one wave) that take half a second."""
    import torch
    torch.cuda._sleep(1000)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    torch.cuda._sleep(1000000)
    torch.cuda.synchronize()
    return int(5e5 / (time.perf_counter() - t0))


@pytest.fixture(scope="module")
def problem():
    isl = synth.star_islands(71, 3, (0.1, 0.2), nodes=64)
    return isl, Curves(isl)


def _busy(spin, call):
    """The result of call() on a side stream beside a spinning null stream
    (which it may still wait for: streams can share a hardware queue)."""
    import torch
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    torch.cuda._sleep(spin)
    with torch.cuda.stream(side):
        out = call()
    torch.cuda.synchronize()
    return out


# eight systems take two work-groups of the step that counts them; a first
# handle leaves its counters in memory that the second may get
# Tolerance: GMRES to 1e-12 of the residual times the matrix' condition
# number (2.8e3), and sqrt(195) from the 2-norm to the largest entry: 4e-8.
def test_first_solve(spin, problem):
    import torch
    from paper_1306_0612_amd import lbs
    isl, cv = problem
    G = np.random.default_rng(72).normal(size=(8, cv.n))
    A = nystrom.system_matrix(cv)
    ref = np.linalg.solve(A, np.concatenate([2 * G, np.zeros((8, cv.m))], 1).T).T
    g = torch.tensor(G.ravel(), device="cuda")
    for _ in range(2):
        sol = lbs.Solver([isl] * 8, graphs=0)
        torch.cuda.synchronize()
        s, a, info = _busy(spin, lambda: sol.solve(g, tol=1e-12, precision="fp64"))
        got = torch.cat([s.reshape(8, -1), a.reshape(8, -1)], 1).cpu().numpy()
        assert np.abs(got - ref).max() < 4e-8 * np.abs(ref).max()
        sol.close()


# Tolerances: those of the operator's parity tests, 1e-10 and 1e-6.
@pytest.mark.parametrize("prec,tol", [("fp64", 1e-10), ("mixed", 1e-6)])
def test_setup_and_first_product(spin, problem, prec, tol):
    import torch
    from paper_1306_0612_amd import lbs
    isl, cv = problem
    X = np.random.default_rng(73).normal(size=(2, cv.n))
    ref = X @ (nystrom.kernel_block(cv, np.arange(cv.n)) + np.eye(cv.n)).T
    x = torch.tensor(X, device="cuda")

    def call():
        sol = lbs.Solver(isl)
        one = sol.matvec(x[0].contiguous(), "iplusk", prec)
        return sol, one, sol.matvec(x, "iplusk", prec)  # two columns: larger buffers

    for _ in range(2):
        sol, one, two = _busy(spin, call)
        for y, r in ((one, ref[0]), (two, ref)):
            assert np.abs(y.cpu().numpy() - r).max() < tol * np.abs(r).max()
        sol.close()
