"""GPU: the launch shapes of a restricted sweep, either side of their lines, against
box-by-box LU solves: the interior boxes' product with two parts or one to a tile
(512 work-groups and more in FP64, 768 in FP32; 8 x 8/2 boxes take four row tiles a
group of sixteen boxes), and the IB boxes' 64-row chunks in four, two or one parts
(until there are 128 work-groups; three chunks a box).

FP64 at 1e-10 per row class (explicit inverses against LU solves), FP32 at 1e-4, as
for every smoother application."""
import numpy as np
import pytest
import scipy.linalg as la
import torch

import workloads as W
from oracle import hierarchy, schwarz
from _parity import assert_classes, level_classes

pytestmark = pytest.mark.gpu

PRECISIONS = [("fp64", 1e-10), ("fp32", 1e-4)]
# N, rings, points each, radii, interior work-groups, row parts of the IB chunks (the
# 512^2 grid's IB boxes are eliminated)
SHAPES = [(384, 1, 1300, 0.36, 0.36, 508, 1), (384, 1, 1300, 0.355, 0.355, 512, 1),
          (512, 4, 1500, 0.15, 0.37, 764, None), (512, 4, 1500, 0.18, 0.33, 768, None),
          (64, 1, 60, 0.15, 0.15, 12, 4), (64, 1, 60, 0.19, 0.19, 12, 2), (64, 1, 60, 0.32, 0.32, 8, 2),
          (64, 1, 60, 0.43, 0.43, 8, 1)]


def _reference(lev, wl, r):
    """z of one sweep: the interior boxes share one matrix, a box's with IB entries
    is its own"""
    L = lev.L.tocsr()
    has_ib = np.zeros(lev.n, dtype=bool)
    has_ib[:2 * wl.N ** 2] = np.diff(lev.T.tocsr().indptr) > 0
    z, shared, inside = np.zeros(lev.n), None, []
    for p in schwarz.patches(wl.N, wl.box, wl.overlap):
        if has_ib[p.idx].any():
            z[p.own_global] = la.solve(L[p.idx][:, p.idx].toarray(), r[p.idx])[p.own_local]
        else:
            if shared is None:
                shared = la.lu_factor(L[p.idx][:, p.idx].toarray())
            inside.append(p)
    y = la.lu_solve(shared, np.stack([r[p.idx] for p in inside], 1))
    for i, p in enumerate(inside):
        z[p.own_global] = y[p.own_local, i]
    return z


@pytest.mark.parametrize("N,rings,points,inner,outer,groups,parts", SHAPES)
def test_sweep_launch_shapes(N, rings, points, inner, outer, groups, parts):
    from paper_1612_02208_amd import StokesIB
    X, S = W.membrane(points, inner) if rings == 1 else W.annulus(rings, points, inner, outer)
    wl = W.Workload("dispatch", N, 6 if N == 384 else 8, 1.0, 0.1, 1e-3, X, S, np.full(len(S), 40.0), box=8, overlap=2)
    lev = hierarchy.build(wl)[-1]
    r = np.random.default_rng(N + points).uniform(-1, 1, lev.n)
    want = _reference(lev, wl, r)
    for precision, tol in PRECISIONS:
        G = StokesIB(wl, precision=precision)
        st = G.stats()["levels"][-1]
        n_int, items = st["boxes"] - st["ib_boxes"], 3 * st["ib_boxes"]
        assert (n_int + 15) // 16 * 4 == groups
        assert parts is None or (1 if items >= 128 else 2 if 2 * items >= 128 else 4) == parts
        z = G.smoother_apply(-1, torch.from_numpy(r).cuda())
        torch.cuda.synchronize()
        assert_classes(z.cpu().numpy(), want, level_classes(lev.N, lev.T), tol, f"{N} {precision}")
        G.close()
