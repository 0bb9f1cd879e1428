"""GPU: which form of the IB term of L_IB w a level takes (explicit rows, or
interpolation, forces and the gather), by its entries, longest face list and
points, where two of the three pull apart; and that the forms agree there to 1e-12
per row class, as every operator form does."""
import numpy as np
import pytest
import torch
from scipy.spatial import cKDTree

import workloads as W
from _parity import assert_classes

pytestmark = pytest.mark.gpu

OPS_TOL = 1e-12


def _annulus(rings, per, tangent=False):
    X, S = W.annulus(rings, per, 0.2, 0.25 if rings == 4 else 0.3)
    wl = W.Workload("annulus", 512, 8, 1.0, 1e-2, 5e-4, X, S, np.full(len(S), 1e3))
    if tangent:
        d = X[S[:, 1]] - X[S[:, 0]]
        wl.spring_model, wl.rest = "tangent", 0.7 * np.hypot(d[:, 0], d[:, 1])
    return wl


def _scattered():
    X = W.random_points(2000, 5)
    near = cKDTree(X).query(X, k=3)[1]
    S = np.concatenate([near[:, [0, 1]], near[:, [0, 2]]]).astype(np.int32)
    return W.Workload("scattered", 512, 8, 1.0, 1e-2, 5e-4, X, S, np.full(len(S), 1e3))


# system and whether the finest level takes the rows
SYSTEMS = {"thick_shell": (lambda: W.paper_case("thick", 512, 1.0, "mu0.01"), True),   # 4.57 M entries, list 40
           "crowded_annulus": (lambda: _annulus(8, 4096), True),                        # 4 M, 51
           "annulus": (lambda: _annulus(4, 2048), True),                                # 2.35 M, 17
           "tangent_annulus": (lambda: _annulus(4, 2048, True), False),                 # 4.59 M, 17
           "scattered": (_scattered, False)}                                            # 3.3 M, 4


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("which", list(SYSTEMS))
def test_form_of_the_finest_level(which, precision, monkeypatch):
    from paper_1612_02208_amd import StokesIB
    make, rows_expected = SYSTEMS[which]
    wl = make()
    w = torch.from_numpy(np.random.default_rng(2).uniform(-1, 1, 3 * wl.N ** 2)).cuda()
    G = StokesIB(wl, precision=precision)
    own = G.apply(w, level=-1).cpu().numpy()
    G.close()
    monkeypatch.setenv("IBMG_NO_IB_ROWS", "1")
    G = StokesIB(wl, precision=precision)
    chain = G.apply(w, level=-1).cpu().numpy()
    G.close()
    assert np.array_equal(own, chain) != rows_expected
    n2 = 2 * wl.N ** 2
    vel = np.arange(3 * wl.N ** 2) < n2
    assert_classes(own, chain, {"vel": vel, "p": ~vel}, OPS_TOL, which)
