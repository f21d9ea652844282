"""Row draws of more rows than one grid dimension has work-items for."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2501_18456_amd import api

pytestmark = pytest.mark.gpu


def test_more_than_2_to_32_row_draws():
    # 1024 equal weights: the row is the top ten bits of the draw's word
    n, seed = (1 << 32) + 1000, (3 << 32) + 11
    rows = api.draw_rows(torch.ones(1024, dtype=torch.float64, device="cuda"), n, seed)
    at = [0, 1 << 31, 1 << 32, n]
    near = np.unique(np.concatenate([np.arange(x - 40, x + 40) for x in at]))
    for k in near[(near >= 0) & (near < n)].tolist():
        word = O.philox4x32_10((k >> 2, 0, 0, 2), (seed & 0xFFFFFFFF, seed >> 32))[k & 3]
        assert int(rows[k]) == int(word) >> 22, k
