"""A configuration's results do not depend on the call that holds it: the same
rows in calls of different sizes (few configurations are shared out over more
wavefronts than many) give the same bits."""
import numpy as np
import pytest
import torch

from workloads import Workload, draw_params, random_sz0_spins

pytestmark = pytest.mark.gpu


def _model(L, K, M, prec):
    from paper_2206_14307_amd import NQS
    w = Workload("order", L=L, n_rbm=K, n_hidden=M, precision=prec, seed=12)
    m = NQS.from_workload(w)
    m.set_params(torch.from_numpy(draw_params(w, std=0.05).reshape(-1)))
    return m


def _rows(L, S):
    sp = random_sz0_spins(L * L, S, 8)
    sp[0] = np.repeat((-1) ** np.arange(L), L)                    # most antiparallel bonds
    sp[1] = np.repeat(np.arange(L) < L // 2, L) * 2 - 1           # fewest
    return torch.from_numpy(sp).cuda()


@pytest.mark.parametrize("M", [8, 16])
def test_e2_4x4_fp64(M):
    m = _model(4, 1, M, "fp64")
    sp = _rows(4, 4100)
    _, ref = m.lanczos_moments(sp)
    for S in (1, 2, 5, 33, 130, 260, 1030, 2100):
        _, e12 = m.lanczos_moments(sp[:S])
        assert torch.equal(e12, ref[:S]), S


@pytest.mark.parametrize("L,M,sizes", [(6, 72, (1, 15, 16, 17, 76, 303, 304, 310)),
                                       (4, 16, (1, 16, 17, 511, 512, 1023, 1024, 1030))])
def test_e2_fp32(L, M, sizes):
    """Across the sizes at which a wavefront's item takes one image tile or several."""
    m = _model(L, 1, M, "fp32")
    sp = _rows(L, sizes[-1])
    _, ref = m.lanczos_moments(sp)
    for S in sizes:
        _, e12 = m.lanczos_moments(sp[:S])
        assert torch.equal(e12, ref[:S]), S


@pytest.mark.parametrize("L,K,M,prec", [(6, 1, 72, "fp32"), (6, 1, 72, "bf16x2"),
                                        (6, 2, 16, "fp32"), (6, 2, 16, "fp64"),
                                        (6, 1, 16, "bf16x2"), (4, 1, 16, "fp64"),
                                        (4, 2, 8, "fp32")])
def test_eloc_fused(L, K, M, prec):
    """The chunk of 2200 is above every size at which bond lists are shared out."""
    from paper_2206_14307_amd.nqs import _ptr, _stream
    m = _model(L, K, M, prec)
    sp = _rows(L, 2200)
    lp, el = m.eloc(sp)
    for S in (1, 2, 3, 7, 16, 37, 56, 57, 113, 128, 129, 300):
        x = sp[:S].contiguous()
        l1, e1 = m.eloc(x)
        assert torch.equal(e1, el[:S]) and torch.equal(l1, lp[:S]), S
        e2 = torch.empty_like(e1)
        assert m.lib.nqs_eloc_noalloc(m._ctx, _ptr(x), S, None, _ptr(e2), _stream()) == 0
        assert torch.equal(e2, e1), S
        assert torch.equal(m.eloc_grad(x)[1], e1), S
        if K > 1:
            assert torch.equal(m.lanczos_moments(x)[1][:, 0], e1), S


@pytest.mark.parametrize("L,K,M,prec", [(6, 1, 144, "fp32"), (6, 4, 40, "bf16x2"),
                                        (6, 5, 32, "fp32"), (8, 1, 136, "bf16x2"),
                                        (8, 3, 48, "fp32"), (10, 1, 136, "fp32"),
                                        (10, 2, 72, "bf16x2"), (10, 4, 40, "fp32")])
def test_eloc_wide(L, K, M, prec):
    """Row 0 has more antiparallel bonds than one walk of the kernel holds."""
    from paper_2206_14307_amd.nqs import _ptr, _stream
    m = _model(L, K, M, prec)
    sp = _rows(L, 2200 * 2 // (L * L))
    lp, el = m.eloc(sp)
    for S in (1, 2, 3, 5, 7, 10, 16, 24, 40, 60, 90):
        if S > sp.shape[0]:
            break
        x = sp[:S].contiguous()
        l1, e1 = m.eloc(x)
        assert torch.equal(e1, el[:S]) and torch.equal(l1, lp[:S]), S
        e2 = torch.empty_like(e1)
        assert m.lib.nqs_eloc_noalloc(m._ctx, _ptr(x), S, None, _ptr(e2), _stream()) == 0
        assert torch.equal(e2, e1), S
        lg, eg, _ = m.eloc_grad(x)
        assert torch.equal(eg, e1) and torch.equal(lg, l1), S
        if S < 4:
            assert torch.equal(m.lanczos_moments(x)[1][:, 0], e1), S
