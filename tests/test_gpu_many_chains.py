"""Heat-bath sweeps of more chains than one grid dimension has work-items for:
chains at the ends and on both sides of every border draw as they would alone."""
import numpy as np
import pytest
import torch

from paper_2501_18456_amd import _lib as B
from paper_2501_18456_amd import api, synth

pytestmark = pytest.mark.gpu

# q = 21: ten chains a wave, 128 a workgroup of 15 waves: 2^32 work-items at 572.7
# million chains
N, L, Q, SEED, SWEEPS = 580_000_007, 2, 21, 5, 2


def _sample(n):
    """Chains at the ends, around 2^21 workgroups and around 2^32 work-items."""
    at = [0, 1 << 21, 128 << 21, (1 << 32) // 960 * 128, 256 << 21, n]
    near = np.concatenate([np.arange(x - 300, x + 300) for x in at])
    return np.unique(near[(near >= 0) & (near < n)])


@pytest.mark.parametrize("form", ["plain", "live"])
def test_more_chains_than_a_grid_dimension_has_work_items(form):
    h, J = (torch.from_numpy(x).cuda() for x in synth.planted_dense(L, Q, seed=4, sigma_J=0.3))
    chains = api.init_chains(N, L, Q, seed=SEED)
    live = N if form == "plain" else N - 1000
    c = _sample(live)
    idx = torch.from_numpy(c).cuda()
    alone = chains[idx].clone()
    last = chains[live:].clone()
    if form == "plain":
        api.gibbs(h, J, chains, sweeps=SWEEPS, seed=SEED, sampler="gather")
    else:
        rec = torch.zeros(N, 3, dtype=torch.int64, device="cuda")
        rec[:, 0] = SEED
        torch.arange(N, out=rec[:, 2])
        n_live = torch.full((1,), live, dtype=torch.int64, device="cuda")
        tick = torch.zeros(1, dtype=torch.int64, device="cuda")
        ws = api.workspace(B.WS_GIBBS, N, L, Q, 0)
        api.sample_tick(h, J, chains, n_live, SWEEPS, rec.view(torch.uint8).view(-1), tick, ws,
                        keep_layout=False)
    api.gibbs_streams(h, J, alone, SWEEPS, api.chain_streams(np.full(len(c), SEED),
                                                             np.zeros(len(c)), c), sampler="gather")
    assert torch.equal(chains[idx], alone)
    assert torch.equal(chains[live:], last)
