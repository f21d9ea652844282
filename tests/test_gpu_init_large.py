"""Chains of more cells than one grid dimension has work-items for: drawn as any others."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2501_18456_amd import api

pytestmark = pytest.mark.gpu


def test_init_of_more_than_2_to_32_cells():
    L, q, seed = 31, 21, (7 << 32) + 9
    N = (1 << 32) // L + 1000
    chains = api.init_chains(N, L, q, seed=seed)
    at = [0, (1 << 31) // L, (1 << 32) // L, N]
    near = np.unique(np.concatenate([np.arange(x - 3, x + 4) for x in at]))
    for c in near[(near >= 0) & (near < N)].tolist():
        words = np.concatenate([O.philox4x32_10((j, 0, c, 1), (seed & 0xFFFFFFFF, seed >> 32))
                                for j in range((L + 3) // 4)])[:L].astype(np.uint64)
        want = (words * np.uint64(q) >> np.uint64(32)).astype(np.int8)
        assert np.array_equal(chains[c].cpu().numpy(), want), c
