"""The FP32 cache-streaming sampler decides several proposals in a pass with the
roundings of one proposal at a time: whole trajectories of 256 chains (520
proposals each, one near-tie in 10^5 decisions falls either way with the last
bit) have the digests recorded from the kernel that decided one proposal in a
pass.  High, middle and low acceptance."""
import hashlib

import pytest
import torch

from helpers import stress_params
from test_gpu_sampler import make
from workloads import Workload, random_sz0_spins

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,M,std,seed,digest", [
    (6, 40, 0.12, 10, "38823b67c78a2150"), (8, 64, 0.1, 9, "3eba21ac59dfca84"),
    (8, 64, 0.1, 14, "b42cd55bcecc93b6"), (8, 64, 0.11, 4, "97b6fa7cb63d7a2c"),
    (8, 64, 0.12, 10, "6a1d35a9ae575770"), (8, 64, 0.3, 19, "f35a5c115dfd4e8f")])
def test_trajectories_of_one_proposal_at_a_time(L, M, std, seed, digest):
    w = Workload("round", L=L, n_hidden=M, precision="fp32", seed=5, is_complex=True)
    m = make(w, stress_params(w, std, 100 + seed))
    state = m.chain_init(torch.from_numpy(random_sz0_spins(w.N, 256, seed)).cuda())
    spins, _, _ = m.sample(state, 8, n_skip=40, n_burn=200, seed=seed)
    assert hashlib.sha256(spins.cpu().numpy().tobytes()).hexdigest()[:16] == digest
