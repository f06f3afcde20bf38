"""Small calls of the fused E_loc kernel, whose bond lists are split over
wavefronts (1 to 8 shares by the number of configurations): the same
configurations inside one large call (no split) give the same result to FP64
rounding of the sums (terms and their FP32 / FP64 products are the same), and
both match the oracle.  Also through nqs_eloc_noalloc."""
import numpy as np
import pytest
import torch

import oracle
from helpers import TOL, max_rel_err
from workloads import Workload, draw_params, random_sz0_spins

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,K,M,prec", [(6, 1, 72, "fp32"), (6, 2, 16, "bf16x2"),
                                        (6, 1, 16, "fp64"), (4, 1, 16, "fp32"), (4, 2, 8, "fp64")])
def test_split_calls(L, K, M, prec):
    from paper_2206_14307_amd import NQS
    from paper_2206_14307_amd.nqs import _ptr, _stream
    w = Workload("split", L=L, n_rbm=K, n_hidden=M, precision=prec, seed=12)
    p = draw_params(w, std=0.05)
    m = NQS.from_workload(w)
    m.set_params(torch.from_numpy(p.reshape(-1)))
    sp = random_sz0_spins(w.N, 300, 8)
    sp[0] = np.repeat((-1) ** np.arange(L), L)                    # most antiparallel bonds
    sp[1] = np.repeat(np.arange(L) < L // 2, L) * 2 - 1           # fewest
    big = torch.from_numpy(np.tile(sp, (10, 1))).cuda()
    lp, el = (x[:300].cpu().numpy() for x in m.eloc(big))
    n = 6
    om = oracle.Model.from_workload(w)
    assert max_rel_err(el[:n], oracle.eloc_direct(om, p, sp[:n])) < TOL[prec]
    for S in (1, 2, 3, 16, 56, 57, 113, 114, 255):
        x = big[:S].contiguous()
        l1, e1 = m.eloc(x)
        e2 = torch.empty_like(e1)
        assert m.lib.nqs_eloc_noalloc(m._ctx, _ptr(x), S, None, _ptr(e2), _stream()) == 0
        assert max_rel_err(e1.cpu().numpy(), el[:S]) < 1e-12
        assert max_rel_err(l1.cpu().numpy(), lp[:S]) < 1e-12
        assert torch.equal(e1, e2)
