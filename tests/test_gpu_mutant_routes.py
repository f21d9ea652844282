"""Single-mutant scans on both sides of every line between their forms: the bits
of a wild type scanned alone, in agreement with plain FP64 sums."""
import pytest
import torch

from paper_2501_18456_amd import api, synth

pytestmark = pytest.mark.gpu


# (block, wild type) pairs: 256 and 258; 64 L; 2048, 4800 of more than 4096 fields;
# 8192 and 12 288 of more than 1600 and of fewer
@pytest.mark.parametrize("L,q,B", [
    (20, 21, 128), (20, 21, 129), (20, 21, 640), (20, 21, 641), (200, 21, 120), (200, 21, 121),
    (200, 21, 282), (200, 21, 283), (80, 21, 1170), (80, 21, 1171), (80, 21, 1755), (80, 21, 1756),
    (130, 3, 4096), (130, 3, 4097), (30, 5, 1921),
])
def test_wild_types_as_alone(L, q, B):
    h, J = (torch.from_numpy(x).cuda() for x in synth.planted_dense(L, q, seed=L, sigma_J=0.05))
    wt = api.init_chains(B, L, q, seed=3)
    dE = api.single_mutant_scan(h, J, wt)
    for b in (0, 1, B // 2, B - 2, B - 1):
        assert torch.equal(api.single_mutant_scan(h, J, wt[b:b + 1].contiguous()), dE[b:b + 1])
    col = torch.arange(L, device="cuda") * q + wt.long()
    H = torch.stack([J[c].double().sum(0) for c in col[:: max(1, B // 50)]]) + h.view(-1).double()
    H = H.view(-1, L, q)
    ref = H.gather(2, wt[:: max(1, B // 50)].long().unsqueeze(2)) - H
    # FP32 sums of L terms, differences of two: 2 (L + 9) roundings of 2^-24
    mag = float(h.abs().max() + L * J.abs().max())
    assert float((dE[:: max(1, B // 50)].view(-1, L, q) - ref).abs().max()) <= 2.0 ** -23 * (L + 9) * mag
