"""Sweeps by free-running waves (a loading wave and LDS counters instead of
barriers) against the oracle, at the edges of their dispatch and layouts."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2501_18456_amd import _lib as B
from paper_2501_18456_amd import api, synth
from tests.trajectory_check import check_chains

pytestmark = pytest.mark.gpu

CHECKED = 48  # chains replayed by the oracle at each end of the launch


# one chunk, two, three and many; whole and ragged last chunks (4, 8, 12 and 16
# positions); chunks of 1 KB blocks that are no multiple of four; site groups 1,
# 2, 4 and 8; 8, 16 and narrow lanes; 4 to 14 waves of chains with two loading,
# 15 with one, 16 (the form with barriers, as for Metropolis of q <= 4 past 400
# sites); a workgroup of one chain
@pytest.mark.parametrize("L,q,N,sampler", [
    (30, 21, 5000, "gather"), (40, 21, 6001, "gather"), (50, 21, 10000, "gather"),
    (60, 21, 30000, "gather"), (41, 32, 7000, "gather"), (49, 25, 12000, "gather"),
    (81, 17, 9000, "gather"), (61, 16, 7500, "gather"), (201, 12, 30000, "gather"),
    (131, 9, 6000, "gather"), (400, 5, 6000, "gather"), (257, 8, 5000, "gather"),
    (12, 21, 6000, "gather"), (13, 4, 3000, "gather"), (60, 16, 30000, "gather"),
    (33, 12, 32768, "gather"), (24, 7, 32000, "metropolis-gather"),
    (401, 4, 8200, "metropolis-gather"), (400, 4, 8200, "metropolis-gather"),
    (30, 21, 20000, "metropolis-gather"), (41, 21, 257, "metropolis-gather"),
    (60, 16, 20000, "metropolis-gather"), (257, 5, 3000, "metropolis-gather"),
    (45, 32, 9000, "metropolis-gather"), (97, 12, 30000, "metropolis-gather"),
])
def test_free_waves_follow_the_oracle(L, q, N, sampler):
    mh = sampler.startswith("metropolis")
    h, J = synth.planted_dense(L, q, seed=90 + L, sigma_J=0.2 if L < 60 else 0.1)
    start = api.init_chains(N, L, q, seed=6)
    chains = start.clone()
    flips = torch.zeros(1, dtype=torch.int64, device="cuda")
    api.gibbs(torch.from_numpy(h).cuda(), torch.from_numpy(J).cuda(), chains, sweeps=2, seed=6,
              sweep_offset=3, beta=0.9, flips=flips, sampler=sampler)
    assert int(flips.item()) >= int((chains != start).sum().item()) > 0
    run = O.metropolis if mh else O.gibbs_range
    n = min(CHECKED, N // 2)
    for c0 in (0, N - n):
        s0 = start[c0:c0 + n].cpu().numpy()
        ref = run(h, J, s0, q=q, sweeps=2, seed=6, sweep_offset=3, beta=0.9, c0=c0)[0]
        check_chains(h, J, s0, chains[c0:c0 + n].cpu().numpy(), ref, q, 2, 6, sweep_offset=3,
                     beta=0.9, metropolis=mh, c0=c0)


def test_free_waves_follow_the_live_count_and_replay_in_a_graph():
    L, q, cap, live = 50, 21, 9000, 5003
    h, J = (torch.from_numpy(x).cuda() for x in synth.planted_dense(L, q, seed=8, sigma_J=0.1))
    start = api.init_chains(cap, L, q, seed=2)
    streams = api.chain_streams(np.full(cap, 2), np.zeros(cap), np.arange(cap))
    n_live = torch.full((1,), live, dtype=torch.int64, device="cuda")
    tick = torch.zeros(1, dtype=torch.int64, device="cuda")
    ws = api.workspace(B.WS_GIBBS, cap, L, q, 0)
    got = start.clone()
    api.sample_tick(h, J, got, n_live, 2, streams, tick, ws, keep_layout=False)
    want = api.gibbs(h, J, start.clone(), sweeps=2, seed=2)
    assert torch.equal(got[:live], want[:live]) and torch.equal(got[live:], start[live:])
    g = torch.cuda.CUDAGraph()
    chains = start.clone()
    ws2 = torch.empty_like(ws)
    with torch.cuda.graph(g):
        api.gibbs(h, J, chains, sweeps=1, seed=2, H_ws=ws2)
    chains.copy_(start)
    eager = start.clone()
    for _ in range(3):  # the captured call takes sweep 0 every time
        g.replay()
        torch.cuda.synchronize()
        eager = api.gibbs(h, J, eager, sweeps=1, seed=2)
        assert torch.equal(chains, eager)
