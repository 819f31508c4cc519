"""Log sources at infinite and zero distance give the logarithm's own limits,
as for the far ends of a squared distance that overflows: G = -inf and +inf
times the strength, never NaN."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def test_limits():
    import torch
    from paper_1306_0612_amd import lbs
    isl = synth.cap_island(n=32)
    sol = lbs.Solver(isl)
    v = np.array([[0.6, 0.0, -0.8], [0.0, 1.0, 0.0]])
    tg = np.array([[0.0, 0.0, -1.0], [np.inf, 0.0, 0.0], [0.0, -1e200, 0.0], [0.6, 0.0, -0.8]])
    gamma = np.array([1.0, 0.25])
    u = torch.zeros(4, dtype=torch.float64, device="cuda")
    dv, dg, dt = (torch.tensor(a, device="cuda") for a in (v, gamma, tg))
    u = sol.vortex_field(u, dv, dg, dt).cpu().numpy()
    d2 = ((tg[0] - v) ** 2).sum(1)
    ref = ((np.log(2.0) - np.log(d2)) / (4 * np.pi)) @ gamma
    assert abs(u[0] - ref) < 1e-15
    assert u[1] == -np.inf and u[2] == -np.inf and u[3] == np.inf
    # and as strengths of the other sign
    w = sol.vortex_field(torch.zeros(4, dtype=torch.float64, device="cuda"), dv, -dg, dt)
    w = w.cpu().numpy()
    assert w[1] == np.inf and w[2] == np.inf and w[3] == -np.inf
    sol.close()
