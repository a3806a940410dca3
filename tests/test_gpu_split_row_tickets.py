"""The split rows' tickets count modulo the row's chunks: after products that
overlapped on one handle (their own results are then unspecified) the next
product alone is whole again."""
import numpy as np
import pytest
import torch

import graphgen as gg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,opts", [(40000, dict(split_len=64)), (300000, dict(split_len=64)),
                                    (60000, dict(split_len=64, lds_stage=1))])
def test_products_after_overlapping_ones(n, opts):
    from paper_1103_2405_amd import TiledMatrix
    rows = 40  # every row split into hundreds of chunks
    rng = np.random.default_rng(n)
    col = np.concatenate([np.sort(rng.choice(n, n // 2, replace=False)) for _ in range(rows)]).astype(np.int32)
    rp = np.concatenate([np.arange(rows + 1) * (n // 2), np.full(n - rows, rows * (n // 2))]).astype(np.int64)
    csr = (n, n, rp, col, gg.uniform_f32(col.size, 4))
    x = torch.from_numpy(gg.uniform_f32(n, 3)).cuda()
    streams = [torch.cuda.Stream() for _ in range(3)]
    with TiledMatrix(csr, **opts) as A:
        want = A.spmv(x)
        ys = [torch.empty(n, device="cuda") for _ in streams]
        torch.cuda.synchronize()
        for _ in range(20):
            for s, y in zip(streams, ys):
                A.spmv(x, y, stream=s)
        torch.cuda.synchronize()
        for _ in range(3):
            y = torch.full((n,), float("nan"), device="cuda")
            assert torch.equal(A.spmv(x, y), want)
