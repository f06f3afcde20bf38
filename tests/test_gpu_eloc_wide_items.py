"""Work items of the wide E_loc kernel: bond lists longer than one walk (row
stripes), empty shares (few antiparallel bonds), 1 to 8 shares by the number of
configurations, more RBMs than the kernel's record holds.  The same
configurations inside one large call (one share each) give the same result to
FP64 rounding of the sums (the terms are the same), and both match the oracle;
nqs_eloc_noalloc and the log amplitudes handed to the gradient agree too."""
import numpy as np
import pytest
import torch

import oracle
from helpers import TOL, max_rel_err
from workloads import Workload, draw_params, random_sz0_spins

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,K,M,prec", [(10, 1, 136, "fp32"), (10, 2, 72, "bf16x2"),
                                        (8, 3, 48, "fp32"), (8, 1, 144, "bf16x2"),
                                        (6, 1, 136, "fp32"), (6, 5, 32, "bf16x2"),
                                        (6, 4, 40, "fp32")])
def test_wide_items(L, K, M, prec):
    from paper_2206_14307_amd import NQS
    from paper_2206_14307_amd.nqs import _ptr, _stream
    w = Workload("wide", L=L, n_rbm=K, n_hidden=M, precision=prec, seed=21)
    p = draw_params(w, std=0.05)
    m = NQS.from_workload(w)
    m.set_params(torch.from_numpy(p.reshape(-1)))
    sp = random_sz0_spins(w.N, 70, 4)
    sp[0] = np.repeat((-1) ** np.arange(L), L)                    # most antiparallel bonds
    sp[1] = np.repeat(np.arange(L) < L // 2, L) * 2 - 1           # fewest
    n_big = -(-2048 // (w.N // 2)) + 70                           # one share per column block
    big = torch.from_numpy(np.tile(sp, (-(-n_big // 70), 1))).cuda()
    lp, el = (x[:70].cpu().numpy() for x in m.eloc(big))
    om = oracle.Model.from_workload(w)
    assert max_rel_err(el[:3], oracle.eloc_direct(om, p, sp[:3])) < TOL[prec]
    for S in (1, 2, 3, 5, 11, 40, 70):
        x = big[:S].contiguous()
        l1, e1 = m.eloc(x)
        e2 = torch.empty_like(e1)
        assert m.lib.nqs_eloc_noalloc(m._ctx, _ptr(x), S, None, _ptr(e2), _stream()) == 0
        assert max_rel_err(e1.cpu().numpy(), el[:S]) < 1e-12
        assert max_rel_err(l1.cpu().numpy(), lp[:S]) < 1e-12
        assert torch.equal(e1, e2)
    lg, eg, O = m.eloc_grad(big[:5].contiguous())
    O1 = m.grad(big[:5].contiguous())
    assert max_rel_err(eg.cpu().numpy(), el[:5]) < 1e-12
    assert max_rel_err(O.cpu().numpy(), O1.cpu().numpy()) < 2e-5
