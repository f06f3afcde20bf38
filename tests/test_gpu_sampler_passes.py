"""The cache-streaming sampler decides several proposals in a pass over the
chains' caches, as many as the acceptance rate and the LDS for their ratios
allow.  Chains with high, middle and low acceptance (passes that follow
acceptances or rejections, with exchanges left pending), with room for four,
three, two and one proposals (by K; FP64 decides one in a pass), across the cache refresh
after 256 proposals and up to a proposal count that leaves a partial pass,
replay the oracle's trajectories; a decision may differ only after a near-tie."""
import numpy as np
import pytest
import torch

import oracle
from helpers import stress_params
from test_gpu_sampler import compare_trajectories, make
from workloads import Workload, random_sz0_spins

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("std", [0.1, 0.2, 0.4])
@pytest.mark.parametrize("L,K,M,prec", [(6, 2, 24, "fp32"), (4, 16, 8, "fp32"), (4, 22, 8, "fp32"),
                                        (4, 40, 8, "fp32"), (4, 1, 24, "fp64"),
                                        (4, 12, 8, "fp64"), (4, 20, 8, "fp64")])
def test_passes_replay(L, K, M, prec, std):
    w = Workload("passes", L=L, n_rbm=K, n_hidden=M, precision=prec, seed=5, is_complex=True)
    p = stress_params(w, std, 21)
    om = oracle.Model.from_workload(w)
    C, n_per, n_skip, n_burn, seed = 5, 13, 3, 270, 77
    init = random_sz0_spins(w.N, C, 8)
    ref, acc_ref, final_ref, ctr_ref, _, log = oracle.exchange_metropolis(
        om, p, init, seed, n_per, n_skip, n_burn, record=True)
    m = make(w, p)
    state = m.chain_init(torch.from_numpy(init).cuda())
    spins, acc, _ = m.sample(state, n_per, n_skip=n_skip, n_burn=n_burn, seed=seed)
    diverged = compare_trajectories(spins.cpu().numpy(), ref, log, n_per,
                                    1e-10 if prec == "fp64" else 2e-5)
    assert diverged <= 1
    st = state.cpu().numpy().view(np.uint64)
    assert (st[:, 2] == ctr_ref.astype(np.uint64)).all()
    if diverged == 0:
        assert np.allclose(acc.cpu().numpy(), acc_ref, atol=1e-6)
        bits = [int(sum(1 << i for i in range(w.N) if f[i] > 0)) for f in final_ref]
        assert st[:, 0].tolist() == bits
