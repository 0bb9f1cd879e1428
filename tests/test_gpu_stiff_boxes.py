"""GPU: the Schwarz boxes' local solves where the structure is far stiffer than
the fluid, against box-by-box LU solves refined in extended precision: boxes
without overlap, small and large ones, whole rows and the eliminated form, and
the paper's thin membrane at its largest stiffness.

An elimination without pivoting that is stable in the ordinary sense leaves a
relative error of a modest multiple of the unit roundoff times the ratio of the
stiffest to the softest velocity mode, at most s = max diag(T) / (rho/dt + 4
mu/h^2) here: 100 eps s per kind of unknown, and no less than 1e-13."""
import numpy as np
import pytest
import scipy.linalg as la
import torch

import workloads as W
from oracle import hierarchy, schwarz

pytestmark = pytest.mark.gpu


def _annulus(N, box, overlap, mu, dt, kappa, rings=2):
    X, S = W.annulus(rings, 3 * N, 0.2, 0.27 if rings == 2 else 0.45)
    return W.Workload("stiff", N, 8, 1.0, mu, dt, X, S, np.full(len(S), kappa), box=box, overlap=overlap)


SYSTEMS = {"no_overlap": lambda: _annulus(64, 8, 0, 1e-3, 1e-2, 1e8),
           "no_overlap_softer": lambda: _annulus(64, 8, 0, 1e-3, 1e-2, 1e5),
           "box_8_2": lambda: _annulus(32, 8, 2, 1e-2, 5e-4, 1e8),
           "box_4_1": lambda: _annulus(32, 4, 1, 1e-3, 1e-2, 1e8),
           "box_16_4": lambda: _annulus(32, 16, 4, 1e-3, 1e-2, 1e8),
           "eliminated": lambda: _annulus(128, 16, 4, 1e-2, 5e-4, 1e8, rings=8),
           "thin_membrane": lambda: W.paper_case("thin", 128, 500.0, "mu0.01", box=16, overlap=4)}


def _refined(A, b):
    lu = la.lu_factor(A)
    A, b = A.astype(np.longdouble), b.astype(np.longdouble)
    x = la.lu_solve(lu, b.astype(float)).astype(np.longdouble)
    for _ in range(6):
        x = x + la.lu_solve(lu, (b - A @ x).astype(float))
    return x.astype(float)


@pytest.mark.parametrize("name", list(SYSTEMS))
def test_stiff_box_solves(name):
    from paper_1612_02208_amd import StokesIB
    wl = SYSTEMS[name]()
    lev = hierarchy.build(wl)[-1]
    L, T, n2 = lev.L.tocsr(), lev.T.tocsr(), 2 * wl.N * wl.N
    r = np.random.default_rng(1).uniform(-1, 1, lev.n)
    G = StokesIB(wl)
    z = G.smoother_apply(-1, torch.from_numpy(r).cuda())
    torch.cuda.synchronize()
    z = z.cpu().numpy()
    G.close()
    has_ib = np.diff(T.indptr) > 0
    boxes = [p for p in schwarz.patches(wl.N, wl.box, wl.overlap) if has_ib[p.idx[p.idx < n2]].any()]
    s = float(T.diagonal().max()) / (wl.rho / wl.dt + 4.0 * wl.mu * wl.N ** 2)
    tol = max(1e-13, 100.0 * np.finfo(float).eps * s)
    for p in boxes[::max(1, len(boxes) // 8)]:
        want = _refined(L[p.idx][:, p.idx].toarray(), r[p.idx])[p.own_local]
        got = z[p.own_global]
        for kind in (p.own_global < n2, p.own_global >= n2):
            err = np.linalg.norm((got - want)[kind]) / np.linalg.norm(want[kind])
            assert err <= tol, (name, err, tol)
