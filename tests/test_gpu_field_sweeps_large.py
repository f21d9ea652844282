"""Field-form sweeps of more chains than one grid dimension has waves for: chains
at the ends and around the border draw as they would alone."""
import numpy as np
import pytest
import torch

from paper_2501_18456_amd import api, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sampler", ["fields", "metropolis-fields"])
def test_field_sweeps_of_more_than_2_to_26_chains(sampler):
    L, q, seed, sweeps, N = 3, 3, 6, 2, (1 << 26) + 1001
    h, J = (torch.from_numpy(x).cuda() for x in synth.planted_dense(L, q, seed=4, sigma_J=0.3))
    chains = api.init_chains(N, L, q, seed=seed)
    at = [0, 1 << 24, 1 << 25, 1 << 26, N]
    near = np.unique(np.concatenate([np.arange(x - 200, x + 200) for x in at]))
    c = near[(near >= 0) & (near < N)]
    idx = torch.from_numpy(c).cuda()
    alone = chains[idx].clone()
    api.gibbs(h, J, chains, sweeps=sweeps, seed=seed, sampler=sampler)
    api.gibbs_streams(h, J, alone, sweeps, api.chain_streams(np.full(len(c), seed),
                                                             np.zeros(len(c)), c), sampler=sampler)
    assert torch.equal(chains[idx], alone)
