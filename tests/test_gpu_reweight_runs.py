"""Sequence weights of alignments large enough that a workgroup takes a run of
several tiles: open pairs listed across tiles, a list that overflows in the middle
of a run with pairs of earlier tiles in it, runs that end in the unpartnered
middle row.  Counts equal a plain one-hot product's and the oracle's."""
import math

import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2501_18456_amd import api

pytestmark = pytest.mark.gpu


def _families(M, L, q, n, g):
    """Rows of n families of equal size, in random order: about 65536 / n open
    pairs in every tile, some similar and some not."""
    base = torch.randint(0, q, (n, L), generator=g, device="cuda", dtype=torch.int8)
    X = base[torch.randint(0, n, (M,), generator=g, device="cuda")]
    rate = 0.35 * torch.rand(M, 1, generator=g, device="cuda")
    mut = torch.rand(M, L, generator=g, device="cuda") < rate
    return torch.where(mut, torch.randint(0, q, (M, L), generator=g, device="cuda",
                                          dtype=torch.int8), X)


def _counts(X, q, theta):
    """N^(m) from the one-hot product (at most L identical positions: exact)."""
    M, L = X.shape
    one = torch.nn.functional.one_hot(X.long(), q).view(M, L * q).half()
    need = math.ceil(theta * L - 1e-6)
    n = torch.empty(M, dtype=torch.int32, device="cuda")
    for m in range(0, M, 4096):
        n[m:m + 4096] = ((one[m:m + 4096] @ one.t()) >= need).sum(1)
    return n


# 98, 99 (runs of 2 tiles), 196 and 197 (of 9) block-rows; codes of three dimensions
# and one; four, two and one rows per thread by planes; `tight` rows of one family in
# the middle of the alignment (their tiles hold more open pairs than the list)
@pytest.mark.parametrize("M,L,q,n,tight", [
    (25_000, 20, 21, 300, 0), (25_300, 20, 4, 120, 700), (25_000, 100, 21, 200, 600),
    (25_200, 40, 21, 1, 0), (50_000, 30, 21, 150, 2000), (50_300, 100, 5, 400, 900),
    (50_300, 130, 21, 250, 1500), (50_000, 200, 21, 90, 3000), (25_300, 300, 21, 200, 800),
])
def test_counts_of_runs_of_tiles(M, L, q, n, tight):
    g = torch.Generator(device="cuda")
    g.manual_seed(M + L)
    X = _families(M, L, q, n, g)
    if tight:
        X[M // 2:M // 2 + tight] = _families(tight, L, q, 1, g)
    got, w, meff = api.reweight(X.contiguous(), q, 0.8)
    assert torch.equal(got, _counts(X, q, 0.8))
    assert torch.equal(w, 1.0 / got.double())
    assert abs(float(meff.item()) - float(w.sum())) <= 1e-12 * float(w.sum())
    rows = np.array([0, 1, 255, 256, M // 2, M // 2 + tight - 1 if tight else M // 3, M - 1])
    assert np.array_equal(got.cpu().numpy()[rows], O.reweight_rows(X.cpu().numpy(), rows, 0.8))
