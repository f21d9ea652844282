"""Energies of more sequences than one launch of 64 per workgroup can number:
every sequence's, on both sides of the launches' borders and of 2^29."""
import pytest
import torch

from paper_2501_18456_amd import _lib, api

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,live", [((1 << 29) + 70, None), ((1 << 29) + 70, (1 << 29) + 65),
                                    ((1 << 30) + 70, None), ((1 << 30) + 70, (1 << 30) + 65)])
def test_energies_of_more_than_2_to_29_sequences(B, live):
    L, q = 2, 4
    g = torch.Generator(device="cuda")
    g.manual_seed(29)
    # multiples of 2^-10: the sums of Eq. (1) are exact, so are the energies
    h = torch.randint(-2048, 2048, (L, q), generator=g, device="cuda").float() / 1024
    block = torch.randint(-2048, 2048, (q, q), generator=g, device="cuda").float() / 1024
    J = torch.zeros(L * q, L * q, device="cuda")
    J[:q, q:], J[q:, :q] = block, block.t()
    X = torch.randint(0, q, (B, L), generator=g, device="cuda", dtype=torch.int8)
    E = torch.full((B,), 99.0, device="cuda")
    ws = api.workspace(_lib.WS_ENERGY, B, L, q, 0)
    if live is None:
        E = api.energy(h, J, X, ws=ws)
    else:
        n = torch.tensor([live], dtype=torch.int64, device="cuda")
        api.energy_batch(h, J, X, n, E, ws)
    ref = -(h[0][:, None] + h[1][None, :] + block).view(-1)
    end = B if live is None else live
    for b in range(0, end, 1 << 26):
        x = X[b:min(b + (1 << 26), end)]
        want = ref[x[:, 0].long() * q + x[:, 1].long()]
        assert torch.equal(E[b:b + len(x)], want), b
    assert bool((E[end:] == 99.0).all())
