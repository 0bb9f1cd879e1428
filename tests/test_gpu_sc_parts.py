"""GPU: the Schur-complement smoother's runs of small colours, one per velocity
component where the springs leave the components apart and one for both where
tangent blocks couple them, against the oracle: components with unequal and empty
colours, colours of more than half a work-group's rows, both precisions.

FP64 at 1e-10 per row class, FP32 at 1e-4, as for every smoother application."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle.solver import Problem
from _parity import assert_classes, level_classes

pytestmark = pytest.mark.gpu


def _system(kind):
    if kind == "line":    # a vertical fibre: the components' rows differ in number
        M = 40
        X = np.stack([np.full(M, 0.37), 0.2 + 0.6 * np.arange(M) / M], 1)
        S = np.stack([np.arange(M - 1), np.arange(1, M)], 1).astype(np.int32)
    elif kind == "dense":
        X, S = W.annulus(2, 300, 0.2, 0.25)
    else:
        X, S = W.membrane(200, 0.25)
    wl = W.Workload(f"sc_{kind}", 64, 8, 0.0, 1.0, 1e-2, X, S, np.full(len(S), 300.0), box=8, overlap=2, smoother="sc")
    if kind == "tangent":
        d = X[S[:, 1]] - X[S[:, 0]]
        wl.spring_model, wl.rest = "tangent", 0.7 * np.hypot(d[:, 0], d[:, 1])
    return wl


@pytest.mark.parametrize("precision,tol", [("fp64", 1e-10), ("fp32", 1e-4)])
@pytest.mark.parametrize("kind", ["line", "ring", "dense", "tangent"])
def test_sc_smoother(kind, precision, tol):
    from paper_1612_02208_amd import StokesIB
    wl = _system(kind)
    P = Problem(wl)
    G = StokesIB(wl, precision=precision)
    rng = np.random.default_rng(4)
    for l in range(1, len(P.levels)):
        lev = P.levels[l]
        r = rng.uniform(-1, 1, lev.n)
        z = G.smoother_apply(l, torch.from_numpy(r).cuda())
        torch.cuda.synchronize()
        assert_classes(z.cpu().numpy(), P.mg.smoothers[l](r), level_classes(lev.N, lev.T), tol, f"level {lev.N}")
    G.close()
