"""Single-mutant scans by a workgroup per (column block, wild type) and by a
wave: the same bits, in agreement with the oracle."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2501_18456_amd import api, synth

pytestmark = pytest.mark.gpu


# fewer sites than eighths, one block and several, ragged last blocks, eighths
# of more than 16 and more than 64 rows, 2 to 32 states, batches on either side
# of the split form's range and of eight rows in flight
@pytest.mark.parametrize("L,q,B", [
    (1, 21, 3), (3, 5, 70), (13, 21, 500), (40, 32, 300), (100, 21, 150), (130, 2, 900),
    (203, 21, 100), (256, 20, 500), (520, 8, 40), (1000, 3, 2),
])
def test_mutants_same_in_every_form(L, q, B):
    h, J = synth.planted_dense(L, q, seed=50 + L, sigma_J=0.05)
    hg, Jg = torch.from_numpy(h).cuda(), torch.from_numpy(J).cuda()
    wt = api.init_chains(B, L, q, seed=3)
    dE = api.single_mutant_scan(hg, Jg, wt)
    for b in (0, B // 2, B - 1):  # alone: the split form
        assert torch.equal(api.single_mutant_scan(hg, Jg, wt[b:b + 1]), dE[b:b + 1])
        w = wt[b].cpu().numpy()
        ref = O.mutant_scan(h, J, w, q)
        # FP32 sums of L terms, differences of two: 2 (L + 9) roundings of 2^-24
        mag = np.abs(h).max() + L * np.abs(J).max()
        assert np.abs(dE[b].cpu().numpy() - ref).max() <= 2.0 ** -23 * (L + 9) * mag
        assert np.all(dE[b].cpu().numpy().reshape(L, q)[np.arange(L), w] == 0)
