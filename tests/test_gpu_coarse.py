"""GPU: the coarsest direct solve at the sizes where its inversion changes
shape (one narrow 128-column step, an exact multiple, a ragged last step, the
largest grid), with and without the velocity null vectors, and with springs
shorter than their rest length (the pivoted elimination), against the oracle's
bordered solve at 1e-10 per row class."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle.solver import Problem
from _parity import assert_classes, level_classes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rho,mu,rest", [(0.0, 1.0, 0.0), (1.0, 1e-2, 0.0), (1.0, 0.1, 1.4), (0.0, 1.0, 0.6)])
@pytest.mark.parametrize("coarse", [4, 5, 8, 13, 16])
def test_coarse_solve(coarse, rho, mu, rest):
    from paper_1612_02208_amd import StokesIB
    X, S = W.membrane(10 * coarse + 1, 0.22, centre=(0.47, 0.52))
    kw = {}
    if rest:
        d = X[S[:, 1]] - X[S[:, 0]]
        kw = dict(spring_model="tangent", rest=rest * np.hypot(d[:, 0], d[:, 1]))
    wl = W.Workload("coarse", 2 * coarse, coarse, rho, mu, 1e-3, X, S, np.full(len(S), 50.0), box=coarse, overlap=1, **kw)
    P = Problem(wl)
    G = StokesIB(wl)
    r = np.random.default_rng(coarse).uniform(-1, 1, P.levels[0].n)
    x = G.coarse_solve(torch.from_numpy(r).cuda())
    torch.cuda.synchronize()
    lev = P.levels[0]
    assert_classes(x.cpu().numpy(), P.mg.coarse(r), level_classes(lev.N, lev.T), 1e-10, "coarse solve")
    G.close()
