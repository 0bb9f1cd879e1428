"""GPU: the residual that the V-cycle restricts after several pre-smoothing
iterations.  An FP32-smoother V-cycle is compared with the FP64 one over 40
right-hand sides: formed as b - L w, the residual holds what rounding did to w,
and the coarse levels take it out again.

The limits are the geometric means of a V-cycle that restricts b - L w (3.5e-7,
4.9e-7 and 7.1e-6 for five, six and seven iterations; standard deviations of
the logarithm 0.9, 1.1 and 2.1) times exp(3 standard errors)."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

LIMITS = [(5, 5.3e-7), (6, 8.1e-7), (7, 1.9e-5)]
N = 128


def _system(nu):
    X, S = W.membrane(4 * N, 0.25)
    return W.Workload("residual_128", N, 8, 1.0, 1e-2, 5e-4, X, S, np.full(len(S), 1e6), nu1=nu, nu2=nu)


def _rhs(count):
    r = torch.stack([torch.from_numpy(W.rhs(N, seed)) for seed in range(count)]).cuda()
    r[:, 2 * N * N:] -= r[:, 2 * N * N:].mean(dim=1, keepdim=True)
    return r


def _mean_error(z, want):
    return float(torch.exp(torch.log((z - want).norm(dim=1) / want.norm(dim=1)).mean()))


@pytest.mark.parametrize("nu,limit", LIMITS)
def test_fp32_vcycle_error(nu, limit):
    from paper_1612_02208_amd import StokesIB
    r = _rhs(40)
    out = {}
    for precision in ("fp64", "fp32"):
        G = StokesIB(_system(nu), precision=precision)
        out[precision] = torch.stack([G.vcycle(x) for x in r])
        torch.cuda.synchronize()
        G.close()
    err = _mean_error(out["fp32"], out["fp64"])
    assert err <= limit, err


def test_fp32_batched_vcycle_error():
    from paper_1612_02208_amd import StokesIB, StokesIBBatch
    nu, limit = LIMITS[1]
    r = _rhs(40)
    G = StokesIB(_system(nu))
    want = torch.stack([G.vcycle(x) for x in r])
    torch.cuda.synchronize()
    G.close()
    B = StokesIBBatch([_system(nu) for _ in range(40)], precision="fp32")
    z = torch.stack(list(B.vcycle(list(r))))
    torch.cuda.synchronize()
    B.close()
    err = _mean_error(z, want)
    assert err <= limit, err
