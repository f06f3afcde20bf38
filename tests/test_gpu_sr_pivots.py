"""nqs_sr_solve with pivots down to 1e-310, whose reciprocals leave the FP64 range:
equal derivatives of few bits in a power of two of samples have an exact mean, so
the system is lambda times the identity and the step exactly zero, for any
lambda > 0."""
import numpy as np
import pytest
import torch

from workloads import Workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("S", [1, 4, 64])
@pytest.mark.parametrize("lam", [1e-300, 1e-305, 1e-310])
def test_tiny_pivots(prec, S, lam):
    from paper_2206_14307_amd import NQS
    m = NQS.from_workload(Workload("sr", L=4, n_hidden=8, precision=prec))
    rng = np.random.default_rng(S)
    o = (rng.integers(-99, 99, (1, m.P)) + 1j * rng.integers(-99, 99, (1, m.P))) / 64
    O = np.repeat(o, S, 0).astype(np.complex128 if prec == "fp64" else np.complex64)
    el = 1e-20 * (rng.normal(size=S) + 1j * rng.normal(size=S))   # eps / lambda stays finite
    d = m.sr_solve(torch.from_numpy(O).cuda(), torch.from_numpy(el).cuda(), lam=lam, dtau=0.02)
    assert not d.cpu().numpy().any()
