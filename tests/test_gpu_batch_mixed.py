"""GPU: a batch level whose members differ in the storage of their IB boxes: one
member's are eliminated, another's are whole rows, so that a sweep runs both forms
and the interior boxes between them.  Against each member's own V-cycle, where a
handle of one system takes the forms that fit it alone (FP64 at 1e-10, the bound of
explicit factors against one another; FP32 at 1e-4, as for every smoother
application)."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

BOX, OVERLAP, N = 16, 4, 128
NLOC, NCHUNK = 2 * 24 * 25 + 24 * 24, 3 * BOX * BOX // 64


def _member(points, radius, centre, kappa):
    X, S = W.membrane(points, radius, centre)
    wl = W.Workload(f"member_{points}", N, 8, 1.0, 1e-2, 5e-4, X, S, np.full(len(S), kappa), box=BOX, overlap=OVERLAP)
    wl.nu1 = wl.nu2 = 2
    return wl


# whole rows by the level's size (both precisions), or (FP32) by their stiffness
MIXES = {"small_beside_large": ((500, 0.3, (0.5, 0.5), 1e3), (20, 0.02, (0.4, 0.4), 1e3), "fp64 fp32"),
         "large_beside_small": ((20, 0.02, (0.4, 0.4), 1e3), (500, 0.3, (0.5, 0.5), 1e3), "fp64 fp32"),
         "stiff_beside_soft": ((500, 0.3, (0.5, 0.5), 1e3), (500, 0.3, (0.5, 0.5), 1e7), "fp32")}


@pytest.mark.parametrize("mix", list(MIXES))
@pytest.mark.parametrize("precision,tol", [("fp64", 1e-10), ("fp32", 1e-4)])
def test_mixed_level(mix, precision, tol):
    from paper_1612_02208_amd import StokesIB, StokesIBBatch
    if precision not in MIXES[mix][2]:
        pytest.skip("FP64 boxes keep their form at any stiffness")
    systems = [_member(*m) for m in MIXES[mix][:2]]
    rng = np.random.default_rng(4)
    r = [torch.from_numpy(rng.uniform(-1, 1, 3 * N * N)).cuda() for _ in systems]
    B = StokesIBBatch(systems, precision=precision)
    z = B.vcycle(r)
    torch.cuda.synchronize()
    rows_bytes = []
    for i, s in enumerate(systems):
        G = StokesIB(s, precision=precision)
        want = G.vcycle(r[i])
        torch.cuda.synchronize()
        rows_bytes.append(len(systems) * G.stats()["levels"][-1]["ib_boxes"] * NCHUNK * 64 * NLOC *
                          (8 if precision == "fp64" else 4))
        err = float((z[i] - want).norm() / want.norm())
        assert err <= tol, (i, s.name, err)
        G.close()
    B.close()
    large = [b >= 192 << 20 for b in rows_bytes]
    assert large == ([True, True] if mix == "stiff_beside_soft" else [mix.startswith("small"), mix.startswith("large")])
