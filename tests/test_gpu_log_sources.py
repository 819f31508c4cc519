"""Log sources summed directly (evaluation with zero densities) at squared
distances from 1e-12 to 4, against extended-precision sums.

Tolerance per target: every squared distance carries three rounded
differences and squares, 4 eps of relative error where |x - c| is of order
one but eps / |x - c| per difference close to a centre, that is an error of
2 eps / |x - c| in its log; the log adds 1 ulp, the product, the sums of M
terms and the constants (M + 8) eps of the sum of the terms' sizes."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu
EPS = 2.0 ** -52


@pytest.mark.parametrize("m", [1, 3, 300])
def test_distances(m):
    import torch
    from paper_1306_0612_amd import lbs
    isl = synth.star_islands(81, m, (0.004, 0.008), nodes=16, gap_factor=1.0)
    rng = np.random.default_rng(82)
    A = rng.normal(size=(2, m))
    # around the first centre at distances 1e-6 .. 2 (the entry point takes
    # any sphere point; the densities are zero), ragged against blocks of 256
    c = isl.center[0]
    d = 10.0 ** rng.uniform(-6, 0, 777)
    v = rng.normal(size=(777, 3))
    v -= np.outer(v @ c, c)
    v /= np.linalg.norm(v, axis=1, keepdims=True)
    tg = np.concatenate([np.cos(d)[:, None] * c + np.sin(d)[:, None] * v, [-c]])
    sol = lbs.Solver(isl, close_eval=0)
    S = torch.zeros((2, int(isl.n.sum())), dtype=torch.float64, device="cuda")
    u = sol.eval(S, torch.tensor(A, device="cuda"), torch.tensor(tg, device="cuda")).cpu().numpy()
    C = np.asarray(isl.center)
    L = np.longdouble
    diff = tg.astype(L)[:, None] - C.astype(L)
    d2 = (diff ** 2).sum(2)
    G = (np.log(L(2)) - np.log(d2)) / (4 * L(np.pi))
    size = np.abs(G) + 0.1
    for r in range(2):
        ref = G @ A[r].astype(L)
        tol = (np.abs(A[r]) * ((m + 10) * EPS * size + 2 * EPS / np.sqrt(d2))).sum(1)
        assert (np.abs(u[r] - ref) < tol).all(), r
    sol.close()
