"""The GMRES loop's wait on the iteration's result in host memory: restarts
(the iteration count starts again with each cycle), one and many systems,
captured and launched iterations, and two threads that solve at once on
their own handles and streams.  Reference: the discrete system itself, its
residual formed by the FP64 operator.

Tolerance: the stopping residual 1e-11 (relative, of the system that GMRES
runs on); its recurrence and the operator add rounding of the order of
1e-13, and the unpreconditioned form is asked for, so the true residual is
that one: 1.1e-11."""
import threading

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("graphs", [0, 1])
@pytest.mark.parametrize("rhs", [1, 6])
def test_restarts_and_threads(graphs, rhs):
    import torch
    from paper_1306_0612_amd import lbs
    isl = [synth.star_islands(87 + q, 5 + q, (0.08, 0.15), nodes=64) for q in range(2)]
    out = [None, None]

    def run(q):
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            sol = lbs.Solver(isl[q], restart=25, graphs=graphs, precond=0)
            n, m = int(isl[q].n.sum()), isl[q].m
            g = torch.tensor(np.random.default_rng(q).normal(size=(rhs, n)), device="cuda")
            worst = 0.0
            for _ in range(3):
                s, a, info = sol.solve(g, tol=1e-11, precision="fp64")
                assert info["iters"] > 25  # more than one cycle
                x = torch.cat([s.reshape(rhs, n), a.reshape(rhs, m)], 1)
                res = sol.matvec(x, "system", "fp64").reshape(rhs, n + m)
                res[:, :n] -= 2.0 * g
                worst = max(worst, float((res.norm(dim=1) / (2.0 * g.norm(dim=1))).max()))
            stream.synchronize()
            sol.close()
        out[q] = worst

    threads = [threading.Thread(target=run, args=(q,)) for q in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert out[0] is not None and out[1] is not None
    assert max(out) < 1.1e-11, out
