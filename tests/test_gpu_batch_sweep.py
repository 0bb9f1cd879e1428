"""GPU: the batched sweep and smoothing step where their forms meet: levels whose
members keep whole rows, are eliminated or do both, a member without a structure
and members of several sizes, for one to three smoothing iterations, against each
member's own single-system V-cycle (FP64 at 1e-10, the bound of explicit factors
against one another; FP32 at 1e-4, as for every smoother application)."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


def _member(N, M, radius, box, overlap, nu, kappa=1e3):
    X, S = W.membrane(M, radius) if M else (np.zeros((0, 2)), np.zeros((0, 2), dtype=np.int32))
    wl = W.Workload(f"member_{N}_{M}", N, 8, 1.0, 1e-2, 5e-4, X, S, np.full(len(S), kappa), box=box, overlap=overlap)
    wl.nu1 = wl.nu2 = nu
    return wl


@pytest.mark.parametrize("precision,tol", [("fp64", 1e-10), ("fp32", 1e-4)])
@pytest.mark.parametrize("box,overlap,nu,sizes", [
    (8, 2, 2, [(64, 200), (32, 100), (64, 0), (16, 40)]),            # whole rows only
    (16, 4, 1, [(128, 500), (128, 40), (64, 250), (128, 0)]),        # large boxes: eliminated beside whole rows
    (8, 2, 3, [(128, 600)] * 12 + [(64, 250)] * 3)])                 # eliminated by their number
def test_batched_vcycle(box, overlap, nu, sizes, precision, tol):
    from paper_1612_02208_amd import StokesIB, StokesIBBatch
    systems = [_member(N, M, 0.2 + 0.01 * (i % 7), box, overlap, nu) for i, (N, M) in enumerate(sizes)]
    rng = np.random.default_rng(len(sizes))
    r = [torch.from_numpy(rng.uniform(-1, 1, 3 * s.N * s.N)).cuda() for s in systems]
    B = StokesIBBatch(systems, precision=precision)
    z = B.vcycle(r)
    torch.cuda.synchronize()
    for i, s in enumerate(systems):
        G = StokesIB(s, precision=precision)
        want = G.vcycle(r[i])
        torch.cuda.synchronize()
        err = float((z[i] - want).norm() / want.norm())
        assert err <= tol, (i, s.name, err)
        G.close()
    B.close()
