"""Sweeps on the routes that the planner's measured lines choose: heat-bath plans
of many waves that keep the barriers draw the bits of chains alone; Metropolis
plans of fewer waves than a plan's least, with token rows an odd number apart,
follow the oracle."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2501_18456_amd import api, synth
from tests.trajectory_check import check_chains

pytestmark = pytest.mark.gpu


# 9, 12, 13 and 15 waves; 8, 4 and 2 site groups; 12, 20 and 28 positions a lane
@pytest.mark.parametrize("L,q,N", [
    (200, 4, 25_600), (150, 3, 17_408), (80, 4, 27_600), (70, 8, 23_552), (100, 5, 30_000),
    (50, 9, 25_601), (40, 12, 30_719),
])
def test_heat_bath_of_many_waves_draws_the_bits_of_few(L, q, N):
    h, J = (torch.from_numpy(x).cuda() for x in synth.planted_dense(L, q, seed=L, sigma_J=0.1))
    chains = api.init_chains(N, L, q, seed=3)
    ids = np.r_[0:150, N // 2:N // 2 + 150, N - 150:N]
    idx = torch.from_numpy(ids).cuda()
    alone = chains[idx].clone()
    api.gibbs(h, J, chains, sweeps=2, seed=3, sweep_offset=5)
    streams = api.chain_streams(np.full(len(ids), 3), np.full(len(ids), 5), ids)
    api.gibbs_streams(h, J, alone, 2, streams)
    assert torch.equal(chains[idx], alone)


# one wave of chains, three for two waves' chains, all; 16 and 8 site groups; token
# rows of 1, 2, 4, 6 and 8 (one more) and odd ones; one round and several
@pytest.mark.parametrize("L,q,N", [
    (512, 4, 40), (512, 2, 1100), (323, 3, 300), (250, 2, 1500), (100, 4, 1024), (60, 2, 2048),
    (17, 4, 2000), (1, 3, 9), (2, 8, 700), (250, 8, 1030), (120, 8, 2048), (33, 5, 2500),
    (401, 6, 257), (120, 4, 25_369), (60, 8, 25_369),
])
def test_metropolis_of_16_lanes_follows_the_oracle(L, q, N):
    h, J = synth.planted_dense(L, q, seed=90 + L, sigma_J=0.2 if L < 60 else 0.1)
    start = api.init_chains(N, L, q, seed=6)
    chains = start.clone()
    api.gibbs(torch.from_numpy(h).cuda(), torch.from_numpy(J).cuda(), chains, sweeps=2, seed=6,
              sweep_offset=3, beta=0.9, sampler="metropolis-gather")
    n = min(32, N)
    for c0 in (0, N - n):
        s0 = start[c0:c0 + n].cpu().numpy()
        ref = O.metropolis(h, J, s0, q=q, sweeps=2, seed=6, sweep_offset=3, beta=0.9, c0=c0)[0]
        check_chains(h, J, s0, chains[c0:c0 + n].cpu().numpy(), ref, q, 2, 6, sweep_offset=3,
                     beta=0.9, metropolis=True, c0=c0)
