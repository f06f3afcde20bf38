"""nqs_sr_solve where the factorisation takes several panels of eight 32-row
blocks (full, partial and single-block last panels) and the FP32 Gram each of
its tile sizes (64 and 96 rows, partial last tiles), against the
parameter-space solve (equal by the push-through identity).  The ridge keeps
the systems well conditioned: FP64 1e-9, FP32 (Gram in FP32) 1e-4."""
import numpy as np
import pytest
import torch

import oracle
from workloads import Workload

pytestmark = pytest.mark.gpu


def _problem(P, S, dtype):
    rng = np.random.default_rng(S)
    cn = lambda *s: rng.normal(size=s) + 1j * rng.normal(size=s)
    O = (0.3 * cn(S, P) + cn(1, P) + 0.2 * cn(S, 5) @ cn(5, P)).astype(dtype)
    return O, -20.0 + cn(S)


@pytest.mark.parametrize("prec,S", [("fp64", 256), ("fp64", 257), ("fp64", 523), ("fp32", 31),
                                    ("fp32", 700), ("fp32", 2100), ("fp32", 2801)])
def test_sr_panels_and_tiles(prec, S):
    from paper_2206_14307_amd import NQS
    m = NQS.from_workload(Workload("sr", L=4, n_hidden=8, precision=prec))
    O, el = _problem(m.P, S, np.complex128 if prec == "fp64" else np.complex64)
    got = m.sr_solve(torch.from_numpy(O).cuda(), torch.from_numpy(el).cuda(), lam=0.05,
                     dtau=0.02).cpu().numpy()
    ref = oracle.sr_param_space(O.astype(np.complex128), el, 0.05, 0.02)
    assert np.linalg.norm(got - ref) < (1e-9 if prec == "fp64" else 1e-4) * np.linalg.norm(ref)
