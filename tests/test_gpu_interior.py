"""GPU: the interior boxes' product in parity classes, against the oracle's
box-by-box LU solves, over the box shapes it takes: odd and even boxes (fixed
points of the reflections), no overlap, boxes that wrap the periodic edges,
fewer boxes than a tile of sixteen and ragged last tiles, both work-group
shapes, additive and multiplicative sweeps, both precisions.

FP64 at 1e-10 per row class (explicit inverses against LU solves), FP32 at
1e-4, as for every smoother application."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle.solver import Problem
from _parity import assert_classes, level_classes

pytestmark = pytest.mark.gpu

#            N, coarse, box, overlap, smoother
SHAPES = [(48, 6, 3, 0, "ras"), (60, 15, 5, 1, "ras"), (56, 7, 7, 2, "rms"), (72, 9, 6, 3, "ras"),
          (64, 8, 4, 1, "rms"), (96, 12, 12, 4, "ras"), (80, 10, 2, 2, "ras"), (144, 9, 6, 2, "ras")]


@pytest.mark.parametrize("precision,tol", [("fp64", 1e-10), ("fp32", 1e-4)])
@pytest.mark.parametrize("N,coarse,box,overlap,smoother", SHAPES)
def test_interior_classes(N, coarse, box, overlap, smoother, precision, tol):
    from paper_1612_02208_amd import StokesIB
    # a small structure near one corner: the other edges' boxes are interior
    X, S = W.membrane(17, 0.05, centre=(0.2, 0.25))
    wl = W.Workload("interior", N, coarse, 1.0, 0.1, 1e-3, X, S, np.full(len(S), 40.0), box=box, overlap=overlap,
                    smoother=smoother)
    P = Problem(wl)
    G = StokesIB(wl, precision=precision)
    st = G.stats()["levels"]
    assert st[-1]["boxes"] > st[-1]["ib_boxes"] > 0
    rng = np.random.default_rng(N + box)
    for l in range(1, len(P.levels)):
        lev = P.levels[l]
        r = rng.uniform(-1, 1, lev.n)
        z = G.smoother_apply(l, torch.from_numpy(r).cuda())
        torch.cuda.synchronize()
        assert_classes(z.cpu().numpy(), P.mg.smoothers[l](r), level_classes(lev.N, lev.T), tol, f"level {lev.N}")
    G.close()
