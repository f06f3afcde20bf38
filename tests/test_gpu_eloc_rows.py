"""E_loc of FP32 models without a register-resident bond kernel (stored-t bond
kernel): every lattice size, one and several RBMs, random configurations and
ordered ones whose antiparallel bonds need more than one pass of bond slots
(stripes: 40 of 64 / 108 of 144 / 192 of 256 / 300 of 400 bonds, against 40, 88,
144 and 224 slots), one and many configurations per call; nqs_eloc_grad of the
same models against its two separate calls."""
import numpy as np
import pytest
import torch

import oracle
from helpers import (TOL, eloc_error_scale, logpsi_error_scale, max_logpsi_err,
                     max_scaled_eloc_err, max_scaled_logpsi_err, stress_params)
from workloads import Workload, draw_params, random_sz0_spins

pytestmark = pytest.mark.gpu


def stripes(L):
    row = np.repeat((-1) ** np.arange(L), L)
    return np.stack([row, -row]).astype(np.int8)


@pytest.mark.parametrize("L,K,M,prec", [(4, 1, 32, "fp32"), (4, 3, 8, "fp32"), (6, 1, 40, "fp32"),
                                        (6, 1, 8, "bf16x2"), (8, 2, 24, "fp32"), (8, 1, 64, "bf16x2"),
                                        (10, 1, 24, "fp32")])
def test_eloc_stored_t(L, K, M, prec):
    from paper_2206_14307_amd import NQS
    w = Workload("rows", L=L, n_rbm=K, n_hidden=M, precision=prec, seed=77)
    sp = np.concatenate([random_sz0_spins(w.N, 6 if L < 10 else 3, 3), stripes(L)])
    for p in (draw_params(w), stress_params(w, 0.1, 4)):
        om = oracle.Model.from_workload(w)
        m = NQS.from_workload(w)
        m.set_params(torch.from_numpy(p.reshape(-1)))
        lp, el = m.eloc(torch.from_numpy(sp).cuda())
        kp, ke = logpsi_error_scale(om, p, sp), eloc_error_scale(om, p, sp)
        ref = oracle.eloc_direct(om, p, sp)
        assert max_scaled_logpsi_err(lp.cpu().numpy(), oracle.logpsi(om, p, sp), kp) < TOL[prec]
        assert max_scaled_eloc_err(el.cpu().numpy(), ref, ke) < TOL[prec]
        one = m.eloc(torch.from_numpy(sp[-1:]).cuda(), want_logpsi=False)
        assert max_scaled_eloc_err(one.cpu().numpy(), ref[-1:], ke[-1:]) < TOL[prec]
        # more configurations than workgroups of the split launch
        many = torch.from_numpy(np.tile(sp, (300, 1))).cuda()
        elm = m.eloc(many, want_logpsi=False).reshape(300, len(sp))
        assert max_scaled_eloc_err(elm.cpu().numpy(), ref[None], ke[None]) < TOL[prec]
        lp2, el2, O = m.eloc_grad(many)
        O1, lp1 = m.grad(many, want_logpsi=True)
        assert max_logpsi_err(lp2.cpu().numpy(), lp1.cpu().numpy()) == 0.0
        assert torch.equal(el2.reshape(300, len(sp)), elm) and torch.equal(O, O1)
