"""GPU: prolongation on large grids, a thread per coarse cell with paired fine
values, against the oracle's matrix: rows of cells that are no multiple of the
work-group, and a fine vector that is not aligned to a pair (one thread per fine
point).  1e-12 relative: sums of at most four rounded products."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import transfer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,coarse", [(2048, 8), (2304, 9)])
def test_prolong_pairs(N, coarse):
    from paper_1612_02208_amd import StokesIB
    wl = W.Workload("plain", N, coarse, 1.0, 1e-2, 5e-4, np.zeros((0, 2)), np.zeros((0, 2), dtype=np.int32),
                    np.zeros(0), box=coarse, overlap=1)
    G = StokesIB(wl)
    rng = np.random.default_rng(N)
    e, w = rng.uniform(-1, 1, 3 * N * N // 4), rng.uniform(-1, 1, 3 * N * N)
    want = w + transfer.prolongation(N // 2) @ e
    for shift in (0, 1):
        buf = torch.zeros(3 * N * N + 1, dtype=torch.float64, device="cuda")
        fine = buf[shift:shift + 3 * N * N]
        fine.copy_(torch.from_numpy(w))
        G.prolong_add(-1, torch.from_numpy(e).cuda(), fine)
        torch.cuda.synchronize()
        err = np.linalg.norm(fine.cpu().numpy() - want) / np.linalg.norm(want)
        assert err <= 1e-12, (shift, err)
    G.close()
