"""The located evaluation at target counts around its work-groups of 64, on
a quadtree whose neighbouring leaves differ by many levels (curves of 8 and
of 600 nodes: a coarser leaf covers several neighbour squares and counts
once), targets crowded into one box or spread over the sphere and beyond the
root square, against the oracle's direct sums.

Tolerance: the FMM's error at p64 = 30, ratio 0.47 at worst: 1.5e-10 of a far
box's share of the field, held to 1e-10 of the whole."""
import numpy as np
import pytest

import synth
from oracle import evaluate
from oracle.geometry import Curves

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("leaf", [4, 40])
def test_target_counts(leaf):
    import torch
    from paper_1306_0612_amd import lbs
    isl = synth.star_islands(71, 8, (0.05, 0.2), nodes=[8, 600, 9, 300, 8, 10, 600, 16],
                             gap_factor=1.0)
    cv = Curves(isl)
    sig = np.stack([synth.random_vector(72, cv.n), synth.random_vector(73, cv.n)])
    A = np.stack([synth.random_vector(74, cv.m), np.zeros(cv.m)])
    spread = synth.sphere_targets(75, 150, isl, far_nodes=1.0)
    th = 10.0 ** np.random.default_rng(76).uniform(-5, -1.5, 20)  # beyond the root square
    pole = np.stack([np.sin(th), np.zeros_like(th), np.cos(th)], 1)
    crowd = spread[:1] + 1e-3 * np.random.default_rng(77).normal(size=(100, 3))
    crowd /= np.linalg.norm(crowd, axis=1, keepdims=True)
    tg = np.concatenate([spread, pole, crowd])
    sol = lbs.Solver(isl, leaf_max=leaf, close_eval=0)
    dev = [torch.tensor(v, device="cuda") for v in (sig, A)]
    ref = np.stack([evaluate.evaluate(cv, sig[r], A[r], tg) for r in range(2)])
    for n in (1, 63, 64, 65, 129, len(tg)):
        sel = np.random.default_rng(n).permutation(len(tg))[:n]
        u = sol.eval(*dev, torch.tensor(tg[sel], device="cuda")).cpu().numpy()
        assert (np.abs(u - ref[:, sel]).max(1) < 1e-10 * np.abs(ref).max(1)).all(), n
    sol.close()
