"""Products of matrices without columns or without entries: every row of y is
zero, for every number of right-hand sides (on both sides of each rule for the
rows of the internal copy of X), with X of no elements (a null pointer)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,m", [(0, 0), (1, 0), (1000, 0), (1000, 7), (7, 7)])
@pytest.mark.parametrize("opts", [{}, {"panels": 2}, {"kernel": "coo"}])
def test_products_are_zero(n, m, opts):
    from paper_1103_2405_amd import TiledMatrix
    csr = (n, m, np.zeros(n + 1, np.int64), np.zeros(0, np.int32), np.zeros(0, np.float32))
    with TiledMatrix(csr, **opts) as A:
        y = torch.full((n,), float("nan"), device="cuda")
        A.spmv(torch.ones(m, device="cuda"), y)
        assert torch.equal(y, torch.zeros_like(y))
        for k in (1, 2, 4, 5, 8, 9, 13, 16, 17, 19, 32, 33, 40, 255, 256):
            Y = torch.full((n, k), float("nan"), device="cuda")
            A.spmm(torch.ones(m, k, device="cuda"), Y)
            assert torch.equal(Y, torch.zeros_like(Y)), k
