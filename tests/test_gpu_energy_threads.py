"""Energies of small batches with one sequence per thread and with several, on both
sides of the number of workgroups that decides: the bits of the form without
sub-ranges, in agreement with plain FP64 sums."""
import pytest
import torch

from paper_2501_18456_amd import api, synth

pytestmark = pytest.mark.gpu


def _up(n):
    return -(-n // 256) * 256


# 2048 workgroups of one sequence per thread and 3072 (512 sites: 1024 sub-ranges);
# four and eight sequences per thread; a last thread with none
@pytest.mark.parametrize("L,q,B", [
    (512, 21, 1024), (512, 21, 1025), (512, 32, 1024), (512, 32, 2048), (300, 26, 1500),
    (512, 5, 512), (512, 5, 513), (400, 9, 2047),
])
def test_energies_on_both_sides(L, q, B):
    h, J = (torch.from_numpy(x).cuda() for x in synth.planted_dense(L, q, seed=L, sigma_J=0.05))
    X = api.init_chains(B, L, q, seed=3)
    E = api.energy(h, J, X)
    steps = sum(min(16 * c + 15, L - 1) for c in range(-(-L // 16)))
    pad = -(-B // 64) * 64
    ws = torch.empty(_up(_up(L * pad) + 8 * min(128, steps // 32) * pad), dtype=torch.uint8,
                     device="cuda")
    assert torch.equal(api.energy(h, J, X, ws=ws), E)  # no room for sub-range sums
    assert torch.equal(api.energy(h, J, X[B - 1:]), E[B - 1:])
    col = (torch.arange(L, device="cuda") * q + X.long())[:: max(1, B // 40)]
    ref = torch.stack([-h.view(-1)[c].double().sum() - J[c][:, c].double().triu(1).sum()
                       for c in col])
    # FP32 sums of 16 terms in an FP64 sum: 16 roundings of 2^-24 of the terms
    mag = float(h.abs().max() * L + J.abs().max() * L * (L - 1) / 2)
    assert float((E[:: max(1, B // 40)] - ref).abs().max()) <= 2.0 ** -20 * mag + 1e-6
