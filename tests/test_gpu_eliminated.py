"""GPU: the IB boxes kept eliminated (W rows and the symmetric owned factor)
against the oracle's box-by-box LU solves, at the sizes where the form's parts
change: whole and ragged 64-row chunks of owned unknowns, no overlap (one
narrow elimination block), one and more column slices, the two- to eight-wide
W rows, additive sweeps and colour ranges of multiplicative ones.

FP64 at 1e-10 per row class (explicit factors against LU solves), FP32 at
1e-4, as for every smoother application."""
import numpy as np
import pytest
import torch
from scipy.spatial import cKDTree

import workloads as W
from oracle.solver import Problem
from _parity import assert_classes, level_classes

pytestmark = pytest.mark.gpu

#            N, coarse, box, overlap, smoother, points, precisions
SHAPES = [(128, 8, 16, 4, "ras", 400, ("fp64", "fp32")),
          (160, 10, 10, 2, "ras", 2000, ("fp64", "fp32")),
          (96, 12, 12, 3, "ras", 400, ("fp64",)),
          (104, 13, 13, 4, "ras", 400, ("fp64",)),
          (128, 8, 16, 0, "ras", 400, ("fp64",)),
          (60, 15, 15, 2, "ras", 200, ()),
          (192, 12, 16, 4, "rms", 900, ("fp64",)),
          (96, 12, 24, 1, "ras", 200, ("fp64", "fp32"))]


@pytest.mark.parametrize("N,coarse,box,overlap,smoother,points,large", SHAPES)
def test_eliminated_boxes(N, coarse, box, overlap, smoother, points, large):
    from paper_1612_02208_amd import StokesIB
    # points everywhere, each tied to its nearest neighbours: every box of the
    # finest level is an IB box
    X = W.random_points(points, N + box)
    S = cKDTree(X).query(X, k=3)[1][:, 1:]
    S = np.stack([np.repeat(np.arange(points), 2), S.ravel()], 1).astype(np.int32)
    wl = W.Workload("eliminated", N, coarse, 1.0, 0.1, 1e-3, X, S, np.full(len(S), 40.0), box=box, overlap=overlap,
                    smoother=smoother)
    P = Problem(wl)
    rng = np.random.default_rng(N + box)
    l = len(P.levels) - 1
    lev = P.levels[l]
    r = rng.uniform(-1, 1, lev.n)
    want = P.mg.smoothers[l](r)
    for precision, tol in (("fp64", 1e-10), ("fp32", 1e-4)):
        G = StokesIB(wl, precision=precision)
        n_ib = G.stats()["levels"][-1]["ib_boxes"]
        m = box + 2 * overlap
        rows = n_ib * -(-3 * box * box // 64) * 64 * (2 * m * (m + 1) + m * m) * (8 if precision == "fp64" else 4)
        # the eliminated form starts at 192 MiB of whole rows a launch (a
        # multiplicative sweep needs at least four colours)
        assert (rows >= (192 << 20) * (4 if smoother == "rms" else 1)) == (precision in large), rows >> 20
        z = G.smoother_apply(l, torch.from_numpy(r).cuda())
        torch.cuda.synchronize()
        assert_classes(z.cpu().numpy(), want, level_classes(lev.N, lev.T), tol, f"{precision} level {lev.N}")
        G.close()


#            N, coarse, box, overlap, points: IB boxes x 64-row chunks per launch
ROWS = [(64, 8, 8, 2, 400),    # 64 x 3: whole chunks
        (48, 6, 8, 2, 250),    # 36 x 3: halves
        (48, 6, 8, 2, 3),      # a few boxes: quarters, beside interior ones
        (60, 15, 5, 1, 900),   # 75 owned unknowns: a ragged last chunk, whole
        (40, 10, 5, 2, 150),   # 64 x 2, larger overlap
        (32, 8, 16, 4, 30)]    # 4 x 12 quarters of the largest rows


@pytest.mark.parametrize("precision,tol", [("fp64", 1e-10), ("fp32", 1e-4)])
@pytest.mark.parametrize("N,coarse,box,overlap,points", ROWS)
def test_whole_rows(N, coarse, box, overlap, points, precision, tol):
    """The boxes that keep whole rows: a chunk's rows whole or split between
    work-groups, in one launch with the interior boxes."""
    from paper_1612_02208_amd import StokesIB
    X = W.random_points(points, N + box)
    S = cKDTree(X).query(X, k=2)[1][:, 1:]
    S = np.stack([np.arange(points), S.ravel()], 1).astype(np.int32)
    wl = W.Workload("rows", N, coarse, 1.0, 0.1, 1e-3, X, S, np.full(len(S), 40.0), box=box, overlap=overlap)
    P = Problem(wl)
    G = StokesIB(wl, precision=precision)
    rng = np.random.default_rng(N + points)
    for l in range(1, len(P.levels)):
        lev = P.levels[l]
        r = rng.uniform(-1, 1, lev.n)
        z = G.smoother_apply(l, torch.from_numpy(r).cuda())
        torch.cuda.synchronize()
        assert_classes(z.cpu().numpy(), P.mg.smoothers[l](r), level_classes(lev.N, lev.T), tol, f"level {lev.N}")
    G.close()
