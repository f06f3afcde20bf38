"""The FP32 Gram of nqs_sr_solve with 64-row tiles and a half tile at the end
(650 samples pad to 672 = 10.5 x 64), against the parameter-space solve (equal by
the push-through identity).  FP32 Gram with this ridge: 1e-4."""
import numpy as np
import pytest
import torch

import oracle
from workloads import Workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S", [90, 650])
def test_half_tile_after_full_ones(S):
    from paper_2206_14307_amd import NQS
    m = NQS.from_workload(Workload("sr", L=4, n_hidden=8, precision="fp32"))
    rng = np.random.default_rng(S)
    cn = lambda *s: rng.normal(size=s) + 1j * rng.normal(size=s)
    O = (0.3 * cn(S, m.P) + cn(1, m.P) + 0.2 * cn(S, 5) @ cn(5, m.P)).astype(np.complex64)
    el = -20.0 + cn(S)
    got = m.sr_solve(torch.from_numpy(O).cuda(), torch.from_numpy(el).cuda(), lam=0.05,
                     dtau=0.02).cpu().numpy()
    ref = oracle.sr_param_space(O.astype(np.complex128), el, 0.05, 0.02)
    assert np.linalg.norm(got - ref) < 1e-4 * np.linalg.norm(ref)
