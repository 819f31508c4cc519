"""The Gram-Schmidt step with more columns than its registers hold and more
chunks than a work-group adds itself, both at once, against a plain GMRES in
torch on the same operator; and iteration counts against the oracle's GMRES
(a second pass without effect would cost iterations, not accuracy).

Tolerances.  The residual after k steps is the minimum over the same Krylov
space whatever orthogonal basis spans it; bases that are orthogonal to
k 2^-52 give it to about k^2 2^-52 |A| |x| / |r|, below 1e-9 here, held to
1e-7 relative.  The stopping test compares that number with the tolerance, so
counts differ by at most one, two with restarts."""
import numpy as np
import pytest

import synth
from oracle import gmres as oracle_gmres
from oracle.geometry import Curves

pytestmark = pytest.mark.gpu


def _gmres(torch, op, b, steps):
    """Residual norm relative to |b| after `steps` steps from zero (two
    passes of classical Gram-Schmidt)."""
    V = torch.zeros((steps + 1, b.numel()), dtype=torch.float64, device="cuda")
    H = torch.zeros((steps + 1, steps), dtype=torch.float64)
    beta = b.norm()
    V[0] = b / beta
    for k in range(steps):
        w = op(V[k])
        for _ in range(2):
            h = V[:k + 1] @ w
            w = w - h @ V[:k + 1]
            H[:k + 1, k] += h.cpu()
        H[k + 1, k] = w.norm().cpu()
        V[k + 1] = w / w.norm()
    e = torch.zeros((steps + 1, 1), dtype=torch.float64)
    e[0] = 1.0
    y = torch.linalg.lstsq(H, e, driver="gelsd").solution
    x = (V[:steps].T @ y.cuda().ravel()) * beta
    return float((b - op(x)).norm() / beta)


@pytest.mark.parametrize("steps", [57, 70])
def test_wide_and_many_chunks(steps):
    import torch
    from paper_1306_0612_amd import lbs
    isl = synth.star_islands(84, 40, (0.05, 0.1), nodes=6600)
    sol = lbs.Solver(isl, leaf_max=64, restart=120, precond=0, max_iter=steps)
    assert sol.n_nodes > 263000
    g = torch.tensor(np.random.default_rng(85).normal(size=sol.n_nodes), device="cuda")
    s, a, info = sol.solve(g, tol=1e-14, precision="fp64", check=False)
    assert info["iters"] == steps
    b = torch.cat([2 * g, torch.zeros(sol.n_islands, dtype=torch.float64, device="cuda")])

    def op(v):
        return sol.matvec(v.contiguous(), "system", "fp64")

    got = float((b - op(torch.cat([s, a]))).norm() / b.norm())
    ref = _gmres(torch, op, b, steps)
    assert abs(got - ref) < 1e-7 * ref, (got, ref)
    sol.close()


@pytest.mark.parametrize("precond,restart", [(0, 120), (1, 50), (1, 9)])
def test_iterations(precond, restart):
    import torch
    from paper_1306_0612_amd import lbs
    isl = synth.star_islands(87, 12, (0.05, 0.15), nodes=[40 + (7 * k) % 31 for k in range(12)])
    cv = Curves(isl)
    g = synth.exact_harmonic(cv.x, isl.center, synth.random_data_coeffs(0, isl))
    ref = oracle_gmres.solve_preconditioned(cv, g, 1e-12, restart, 2000, bool(precond))[2]
    sol = lbs.Solver(isl, leaf_max=24, restart=restart, precond=precond, max_iter=2000, p64=48)
    it = sol.solve(torch.tensor(g, device="cuda"), tol=1e-12, precision="fp64")[2]["iters"]
    assert abs(it - ref) <= (1 if restart > it else 2), (it, ref)
    sol.close()
