"""The Gram-Schmidt kernels of the GMRES step over their launch shapes
(columns in registers, chunks folded or reduced by a launch of their own,
several systems) against the dense solve of the oracle.

Tolerance: GMRES stops at a relative residual of 1e-12; the error in the
2-norm is at most the condition number (1.7e3 for the matrix here) times
that, and relative to the largest entry at most sqrt(1671) = 41 times more:
7e-8."""
import numpy as np
import pytest

import synth
from oracle import nystrom
from oracle.geometry import Curves

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_1306_0612_amd import lbs
    lbs.load()
    return torch, lbs


@pytest.fixture(scope="module")
def problem():
    m = 30
    isl = synth.star_islands(87, m, (0.05, 0.15), nodes=[40 + (7 * k) % 31 for k in range(m)])
    cv = Curves(isl)
    A = nystrom.system_matrix(cv)
    G = np.stack([synth.exact_harmonic(cv.x, isl.center, synth.random_data_coeffs(r, isl))
                  for r in range(3)])
    Z = np.linalg.solve(A, np.concatenate([2 * G, np.zeros((3, m))], axis=1).T).T
    return isl, cv, G, Z


# Without the preconditioner this needs 89 Arnoldi columns: restart 120 runs
# every register width and the form above them, 50 restarts on the way; 9
# restarts the preconditioned solve (without it GMRES(9) stagnates).
@pytest.mark.parametrize("precond,restart", [(0, 50), (0, 120), (1, 9), (1, 50)])
@pytest.mark.parametrize("cols", [1, 3])
def test_solution_over_restarts(env, problem, restart, precond, cols):
    torch, lbs = env
    isl, cv, G, Z = problem
    sol = lbs.Solver(isl, leaf_max=24, restart=restart, precond=precond, max_iter=2000)
    s, a, info = sol.solve(torch.tensor(G[:cols], device="cuda"), tol=1e-12, precision="fp64")
    if precond == 0 and restart == 120:
        assert info["iters"] > 56
    s = s.cpu().numpy()
    assert np.abs(s - Z[:cols, :cv.n]).max() / np.abs(Z).max() < 7e-8


def test_batch_of_uneven_geometries(env, problem):
    torch, lbs = env
    isl, cv, G, Z = problem
    other = synth.star_islands(83, 2, (0.1, 0.3), nodes=[33, 48])
    co = Curves(other)
    go = synth.exact_harmonic(co.x, other.center, synth.random_data_coeffs(4, other))
    zo, _ = nystrom.solve_dense(co, go)
    sol = lbs.Solver([other, isl, other], leaf_max=24)
    g = np.concatenate([go, G[0], go])
    for prec in ("fp64", "mixed"):
        s = sol.solve(torch.tensor(np.stack([g, 2 * g]), device="cuda"), tol=1e-12,
                      precision=prec)[0].cpu().numpy()
        no = sol.node_offsets
        for r in range(2):
            for q, ref in ((0, zo), (1, Z[0, :cv.n]), (2, zo)):
                d = s[r, no[q]:no[q + 1]] - (r + 1) * ref
                assert np.abs(d).max() / np.abs(ref).max() < 7e-8, (prec, r, q)


def test_many_chunks(env):
    """Over 256 chunks (262144 unknowns): the partial sums take a launch of
    their own; the solved u against the exact harmonic function (1e-9: ten
    times what the solves at 1e-12 of 1.02M nodes leave)."""
    torch, lbs = env
    isl = synth.star_islands(84, 40, (0.05, 0.1), nodes=6600)
    sol = lbs.Solver(isl, leaf_max=64)
    assert sol.n_nodes > 263000
    coeffs = synth.random_data_coeffs(85, isl)
    xyz = sol.nodes().cpu().numpy()
    g = torch.tensor(synth.exact_harmonic(xyz, isl.center, coeffs), device="cuda")
    tg = synth.sphere_targets(86, 200, isl)
    exact = synth.exact_harmonic(tg, isl.center, coeffs)
    for prec in ("fp64", "mixed"):
        s, a, info = sol.solve(g, tol=1e-12, precision=prec)
        u = sol.eval(s, a, torch.tensor(tg, device="cuda")).cpu().numpy()
        assert np.abs(u - exact).max() / np.abs(exact).max() < 1e-9, prec
