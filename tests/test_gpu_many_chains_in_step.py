"""The form with waves in step at more chains than one grid dimension has work-items
for (16 waves hold 128 chains, 64 of Metropolis at q <= 8): chains at the ends and
on both sides of every border draw as they would alone."""
import numpy as np
import pytest
import torch

from paper_2501_18456_amd import _lib as B
from paper_2501_18456_amd import api, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("q,N,sampler,live", [
    (4, (1 << 28) + 70_000, "metropolis-gather", None), (8, (1 << 29) + 70_000, "gather", None),
    (8, (1 << 29) + 70_000, "gather", (1 << 29) + 69_000)])
def test_more_chains_in_step_than_a_grid_dimension_has_work_items(q, N, sampler, live):
    L, seed, sweeps = 2, 5, 2
    h, J = (torch.from_numpy(x).cuda() for x in synth.planted_dense(L, q, seed=4, sigma_J=0.3))
    chains = api.init_chains(N, L, q, seed=seed)
    n = N if live is None else live
    at = [0, 70_000, 1 << 21, 128 << 21, n]
    near = np.unique(np.concatenate([np.arange(x - 300, x + 300) for x in at]))
    c = near[(near >= 0) & (near < n)]
    idx = torch.from_numpy(c).cuda()
    alone, last = chains[idx].clone(), chains[n:].clone()
    if live is None:
        api.gibbs(h, J, chains, sweeps=sweeps, seed=seed, sampler=sampler)
    else:
        rec = torch.zeros(N, 3, dtype=torch.int64, device="cuda")
        rec[:, 0] = seed
        torch.arange(N, out=rec[:, 2])
        n_live = torch.full((1,), live, dtype=torch.int64, device="cuda")
        ws = api.workspace(B.WS_GIBBS, N, L, q, 0)
        api.sample_tick(h, J, chains, n_live, sweeps, rec.view(torch.uint8).view(-1),
                        torch.zeros(1, dtype=torch.int64, device="cuda"), ws, keep_layout=False)
    api.gibbs_streams(h, J, alone, sweeps, api.chain_streams(np.full(len(c), seed),
                                                             np.zeros(len(c)), c), sampler=sampler)
    assert torch.equal(chains[idx], alone)
    assert torch.equal(chains[n:], last)
