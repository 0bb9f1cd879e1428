"""GPU: the two forms of the IB term of L_IB w (explicit Galerkin rows in the
operator's launch; interpolation, spring forces and the gather) on every
level, the residual-carrying V-cycle included.

Both are sums of at most a few thousand rounded products per row (coarse rows
couple to every face of the level), so they agree, and agree with the
oracle's assembled operator, to 1e-12 per row class like every other operator
check."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle.solver import Problem
from _parity import assert_classes, level_classes

pytestmark = pytest.mark.gpu

OPS_TOL = 1e-12


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float64)).cuda()


def host(t):
    torch.cuda.synchronize()
    return t.detach().cpu().numpy()


def _system(which):
    if which == "one_spring":       # two points, one spring: a handful of rows
        return W.Workload(which, 16, 4, 0.0, 1.0, 1e-2, np.array([[0.51, 0.5], [0.99, 0.01]]),
                          np.array([[0, 1]], dtype=np.int32), np.array([30.0]), box=4, overlap=1)
    if which == "crowded":          # thousands of points on 24^2: rows of a wave each
        X, S = W.annulus(8, 300, 0.1, 0.3)
        return W.Workload(which, 24, 6, 1.0, 0.1, 1e-3, X, S, np.full(len(S), 1e3), box=6, overlap=1)
    X, S = W.membrane(151, 0.27)    # ragged: 16 lanes a row, a last row group that is not full
    d = X[S[:, 1]] - X[S[:, 0]]
    return W.Workload(which, 56, 7, 0.0, 1.0, 1e-3, X, S, np.full(len(S), 1e3), box=7, overlap=2,
                      spring_model="tangent", rest=0.7 * np.hypot(d[:, 0], d[:, 1]))


@pytest.mark.parametrize("which", ["one_spring", "crowded", "ragged_tangent"])
def test_ib_forms_agree_with_the_oracle(which, monkeypatch):
    from paper_1612_02208_amd import StokesIB
    wl = _system(which)
    P = Problem(wl)
    rows = StokesIB(wl)
    monkeypatch.setenv("IBMG_NO_IB_ROWS", "1")
    chain = StokesIB(wl)
    monkeypatch.delenv("IBMG_NO_IB_ROWS")
    rng = np.random.default_rng(3)
    for l, lev in enumerate(P.levels):
        w = rng.uniform(-1, 1, lev.n)
        cl = level_classes(lev.N, lev.T)
        for g, name in ((rows, "rows"), (chain, "chain")):
            assert_classes(host(g.apply(dev(w), level=l)), lev.L @ w, cl, OPS_TOL, f"{name} level {l}")
            assert_classes(host(g.apply(dev(w), level=l, transpose=True)), lev.L.T @ w, cl, OPS_TOL,
                           f"{name} transposed level {l}")
    r = P.project(W.rhs(wl.N, 5))
    cl = level_classes(P.fine.N, P.fine.T)
    for g in (rows, chain):
        assert_classes(host(g.vcycle(dev(r))), P.mg.vcycle(r), cl, 1e-10, "V-cycle")
    rows.close()
    chain.close()
