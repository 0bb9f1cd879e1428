"""GPU: the outer solve's long reductions where their partial sums are read by the
next kernel's blocks (up to 704 of them) and where one block folds them first:
solves of 18 to 30 basis vectors a cycle, checked through the true residual under
the oracle's operator.  The recurrence's residual and the true one differ by
rounding, about 1e-14 of the initial residual a step: the solve's tolerance is met
within 1 %."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import ib, mac

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,coarse,blocks", [(288, 9, 243), (320, 10, 300), (480, 15, 675), (512, 8, 768)])
def test_outer_reductions(N, coarse, blocks):
    from paper_1612_02208_amd import StokesIB
    assert -(-3 * N * N // 1024) == blocks
    X, S = W.membrane(2 * N, 0.25)
    wl = W.Workload("fold", N, coarse, 1.0, 1e-2, 5e-4, X, S, np.full(len(S), 1e3), box=coarse, overlap=2)
    A = mac.momentum(N, wl.rho, wl.mu, wl.dt) + ib.ib_term(X, S, wl.kappa, N, wl.dt)
    L = mac.stokes_ib(A.tocsr(), mac.gradient(N), mac.divergence(N)).tocsr()
    b = W.rhs(N, 5)
    G = StokesIB(wl)
    x, info = G.solve(torch.from_numpy(b).cuda(), rtol=1e-10, restart=30, max_it=120)
    torch.cuda.synchronize()
    x = x.cpu().numpy()
    G.close()
    assert info["converged"], info
    r = b - L @ x
    r[2 * N * N:] -= r[2 * N * N:].mean()
    assert np.linalg.norm(r) <= 1.01e-10 * np.linalg.norm(b), (N, info["iterations"], np.linalg.norm(r) / np.linalg.norm(b))
