"""Energies by a workgroup per range and by one per sub-range (small batches
with room for the sums): the same bits, in agreement with the oracle."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2501_18456_amd import api, synth

pytestmark = pytest.mark.gpu


def _up(n):
    return -(-n // 256) * 256


def _range_bytes(B, L):
    """Workspace that holds the transposed tokens and one sum per range."""
    steps = sum(min(16 * c + 15, L - 1) for c in range(-(-L // 16)))
    parts = min(128, max(1, steps // 32)) if steps else 0
    pad = -(-B // 64) * 64
    return _up(_up(L * pad) + 8 * parts * pad)


# no step, fewer steps than sub-ranges, one range, several, most; one and
# several sequences per thread, whole and partial workgroups
@pytest.mark.parametrize("L,q,B", [
    (1, 21, 5), (2, 4, 3), (5, 21, 65), (16, 21, 64), (17, 5, 1), (33, 32, 300), (50, 8, 2049),
    (64, 26, 513), (123, 21, 1003), (130, 9, 2048), (200, 21, 2050), (300, 3, 4100),
    (40, 25, 9000),
])
def test_energy_same_by_ranges_and_sub_ranges(L, q, B):
    h, J = synth.planted_dense(L, q, seed=30 + L, sigma_J=0.1)
    X = api.init_chains(B, L, q, seed=12)
    hg, Jg = torch.from_numpy(h).cuda(), torch.from_numpy(J).cuda()
    E = api.energy(hg, Jg, X)
    # a workspace with no room for sub-range sums still serves, same bits
    ws = torch.empty(_range_bytes(B, L), dtype=torch.uint8, device="cuda")
    assert torch.equal(api.energy(hg, Jg, X, ws=ws), E)
    # as does one sequence alone
    assert torch.equal(api.energy(hg, Jg, X[B - 1:]), E[B - 1:])
    n = min(B, 64)
    ref = O.energy(h, J, X[:n].cpu().numpy(), q)
    # FP32 sums of 16 terms in an FP64 sum: 16 roundings of 2^-24 of the terms
    mag = np.abs(h).max() * L + np.abs(J).max() * L * (L - 1) / 2
    assert np.abs(E[:n].cpu().numpy() - ref).max() <= 2.0 ** -20 * mag + 1e-6
