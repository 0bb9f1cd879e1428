"""GPU: the FGMRES smoothing step at every length the library takes (one to
eight iterations, each its own kernel instance), its residual taken from the
Arnoldi relation inside the V-cycle, and its breakdown on a zero residual.

FP64 results are compared with the oracle (normalised basis, classical
Gram-Schmidt twice, the residual by an operator application) at 1e-10 per row
class, the bound of every solve-type call; FP32-smoother handles at 1e-4."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle.solver import Problem
from _parity import assert_classes, level_classes

pytestmark = pytest.mark.gpu


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float64)).cuda()


def host(t):
    torch.cuda.synchronize()
    return t.detach().cpu().numpy()


def _system(nu1, nu2):
    # 40^2 -> 20^2 -> 10^2 -> 5^2: a 10^2 grid's last reduction block is nearly empty
    X, S = W.membrane(97, 0.23)
    return W.Workload("smoothing_40", 40, 5, 1.0, 0.1, 1e-3, X, S, np.full(len(S), 2e2), box=5, overlap=1,
                      nu1=nu1, nu2=nu2)


@pytest.mark.parametrize("precision,tol", [("fp64", 1e-10), ("fp32", 1e-4)])
@pytest.mark.parametrize("nu1,nu2", [(1, 2), (3, 4), (5, 1), (6, 7), (8, 3)])
def test_smoothing_lengths(nu1, nu2, precision, tol):
    from paper_1612_02208_amd import StokesIB
    wl = _system(nu1, nu2)
    P = Problem(wl)
    G = StokesIB(wl, precision=precision)
    rng = np.random.default_rng(10 * nu1 + nu2)
    for l in range(1, len(P.levels)):
        lev = P.levels[l]
        w, b = rng.uniform(-1, 1, lev.n), rng.uniform(-1, 1, lev.n)
        out = host(G.smooth(l, dev(w), dev(b), max(nu1, nu2)))
        assert_classes(out, P.mg.smooth(l, w, b, max(nu1, nu2)), level_classes(lev.N, lev.T), tol, f"smooth level {l}")
    r = P.project(W.rhs(wl.N, 4))
    assert_classes(host(G.vcycle(dev(r))), P.mg.vcycle(r), level_classes(P.fine.N, P.fine.T), tol, "V-cycle")
    z = host(G.vcycle(dev(np.zeros(P.fine.n))))
    assert np.all(z == 0.0)          # a zero residual breaks the basis down at once
    r[7] = np.nan
    assert np.isnan(host(G.vcycle(dev(r)))).any()   # and a NaN is not hidden
    G.close()
