"""TILE-COO around its interval of 512 entries: whole intervals are read four
entries a load from any boundary, the last one entry by entry; tiles that begin
at odd offsets, rows that cross intervals, against the oracle."""
import numpy as np
import pytest
import torch

import graphgen as gg
import oracle

pytestmark = pytest.mark.gpu

TOL = 1e-5  # of (|A||x|)_i: FP64 row sums rounded once a tile


@pytest.mark.parametrize("nnz", [1, 511, 512, 513, 1023, 1024, 2049, 70001])
@pytest.mark.parametrize("n_rows", [1, 7, 5000])
@pytest.mark.parametrize("opts", [dict(), dict(tile_width=64), dict(tile_width=256)])
def test_intervals(nnz, n_rows, opts):
    from paper_1103_2405_amd import TiledMatrix
    n_cols = 901
    rng = np.random.RandomState(nnz + n_rows)
    r, c = rng.randint(0, n_rows, nnz), (rng.rand(nnz) ** 2 * n_cols).astype(np.int64)
    order = np.lexsort((c, r))
    rp = np.zeros(n_rows + 1, np.int64)
    np.add.at(rp, r + 1, 1)
    csr = (n_rows, n_cols, np.cumsum(rp), c[order].astype(np.int32), gg.uniform_f32(nnz, 4))
    x = gg.uniform_f32(n_cols, 3)
    tiles = 1 + n_cols // opts.get("tile_width", n_cols)
    bound = tiles * TOL * oracle.absmv(csr, x)
    with TiledMatrix(csr, kernel="coo", relabel=0, **opts) as A:
        y = torch.full((n_rows,), float("nan"), device="cuda")
        A.spmv(torch.from_numpy(x).cuda(), y)
        first = y.clone()
        assert np.all(np.abs(y.cpu().numpy().astype(np.float64) - oracle.spmv(csr, x)) <= bound)
        assert torch.equal(A.spmv(torch.from_numpy(x).cuda()), first)
