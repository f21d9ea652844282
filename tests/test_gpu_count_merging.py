"""Direct chain counts of q <= 8 on both sides of the length from which a bin that
a thread's chains share is added to once: equal to the one-hot products' counts."""
import numpy as np
import pytest
import torch

from paper_2501_18456_amd import _lib as B
from paper_2501_18456_amd import api

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L", [32, 33, 47])
@pytest.mark.parametrize("q,N", [(2, 1027), (5, 1003), (8, 2049)])
@pytest.mark.parametrize("kept", [0.0, 0.6, 1.0])
def test_counts_equal_products(L, q, N, kept):
    g = torch.Generator().manual_seed(q * 100 + L)
    common = torch.randint(0, q, (1, L), generator=g)
    chains = torch.where(torch.rand(N, L, generator=g) < kept, common,
                         torch.randint(0, q, (N, L), generator=g)).to(torch.int8)
    f1 = torch.rand(L * q, generator=g, dtype=torch.float64).cuda()
    f2 = torch.rand((L * q) ** 2, generator=g, dtype=torch.float64).cuda()
    outs = []
    for prec in (B.PREC_FP32, B.PREC_FP32 | B.COUNTS_PRODUCT):
        h, J = torch.zeros(L, q).cuda(), torch.zeros(L * q, L * q).cuda()
        api.train_step(h, J, chains.cuda(), f1, f2, 0.05, 0, 1, 0, prec=prec)  # no sweep
        outs.append((h.cpu().numpy(), J.cpu().numpy()))
    assert np.array_equal(outs[0][0], outs[1][0]) and np.array_equal(outs[0][1], outs[1][1])
