"""Row gathers of more cells than one grid dimension has work-items for."""
import pytest
import torch

from paper_2501_18456_amd import api

pytestmark = pytest.mark.gpu


def test_row_gather_of_more_than_2_to_32_cells():
    M, L, n = 1000, 40, (1 << 32) // 40 + 5000
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    X = torch.randint(0, 21, (M, L), generator=g, device="cuda", dtype=torch.int8)
    rows = torch.randint(0, M, (n,), generator=g, device="cuda", dtype=torch.int32)
    out = api.gather_rows(X, rows)
    for k in range(0, n, 1 << 24):
        r = rows[k:k + (1 << 24)].long()
        assert torch.equal(out[k:k + len(r)], X[r]), k
