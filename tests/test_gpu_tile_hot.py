"""The tile kernel that stages a tile's hottest columns in LDS against the
kernel that gathers every column through the caches: the same bits, product
and fused updates, at the edges of the staged width, and the oracle's bound."""
import numpy as np
import pytest
import torch

import graphgen as gg
import oracle

pytestmark = pytest.mark.gpu

TOL = 1e-5  # of (|A||x|)_i: FP64 row sums rounded once per tile, far inside it


def skewed(n, nnz, seed):
    """Square CSR with skewed columns and row lengths from 0 to a few thousand."""
    rng = np.random.default_rng(seed)
    r = np.concatenate([rng.integers(0, n, nnz // 2), (rng.random(nnz // 2) ** 6 * n).astype(np.int64)])
    c = (rng.random(r.size) ** 3 * n).astype(np.int64)
    key = np.unique(r * n + c)
    rp = np.zeros(n + 1, np.int64)
    np.add.at(rp, key // n + 1, 1)
    return n, n, np.cumsum(rp), (key % n).astype(np.int32), rng.random(key.size, dtype=np.float32)


# staged width 40896: all columns staged, one left over, many left over; one
# and several tiles; the slice counts; workload sizes from a few rows to wide
@pytest.mark.parametrize("n,bounds,wl,S", [(40895, None, 512, 0), (40896, None, None, 1), (40897, None, 96, 2),
                                           (65537, None, 4096, 4), (70001, [5, 45000], 640, 0),
                                           (70001, [66000], 8192, 8)])
def test_staged_hot_columns(n, bounds, wl, S):
    from paper_1103_2405_amd import TiledMatrix
    csr = skewed(n, 6 * n, n)
    x = gg.uniform_f32(n + 1, 7)
    xd = torch.from_numpy(x).cuda()
    got = []
    for stage in (1, -1):
        with TiledMatrix(csr, wl=wl, tile_bounds=bounds, slices=S, lds_stage=stage) as A:
            y = [torch.full((n,), float("nan"), device="cuda") for _ in range(2)]
            A.spmv_internal(xd[:n], y[0])
            A.spmv_internal(xd[1:], y[1])  # 4-byte aligned only
            got.append((A.spmv(xd[:n]), *y, A.pagerank(0.85, 0.0, 6)[0], A.rwr([n // 2], 0.85, 0.0, 6)[0]))
    for a, b in zip(*got):
        assert torch.equal(a, b)
    yh = got[0][0].cpu().numpy().astype(np.float64)
    assert np.all(np.abs(yh - oracle.spmv(csr, x[:n])) <= TOL * oracle.absmv(csr, x[:n]))


def test_large_tile_is_staged_by_default():
    # above the size from which the staged kernel is the default
    from paper_1103_2405_amd import TiledMatrix
    csr = gg.rwr_matrix(gg.rmat(17, 16, seed=3))
    assert csr[3].size > 3 << 20
    x = torch.from_numpy(gg.uniform_f32(csr[1], 5)).cuda()
    with TiledMatrix(csr) as A, TiledMatrix(csr, lds_stage=-1) as B:
        assert torch.equal(A.spmv(x), B.spmv(x))
        assert torch.equal(A.rwr([11], 0.85, 0.0, 7)[0], B.rwr([11], 0.85, 0.0, 7)[0])
