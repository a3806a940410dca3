"""SpMM over the numbers of right-hand sides at which its lanes, passes and
overlaps change, on row-major, column-major (one column, two or three, more) and
split-row workloads, one and several tiles, against the oracle; X may hold
infinities where no entry reads them."""
import numpy as np
import pytest
import torch

import graphgen as gg
import oracle

pytestmark = pytest.mark.gpu

TOL = 1e-5  # of (|A||x|)_i per column: FP64 sums rounded once per tile


@pytest.mark.parametrize("opts", [dict(wl=256, split_len=128), dict(tile_width=700, wl=96, split_len=64),
                                  dict(wl=4096, split_len=1000, wave=32)])
@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 9, 17, 32, 37, 256])
def test_widths(k, opts):
    from paper_1103_2405_amd import TiledMatrix
    rng = np.random.default_rng(k)
    n, m = 2003, 1501
    cols = [[] for _ in range(n)]
    cols[0] = range(1400)  # split
    for r in range(1, n):  # every length from 0 up, most of them short
        cols[r] = np.sort(rng.choice(m - 1, int(rng.integers(0, 3) if r % 3 else rng.integers(0, 150)), replace=False))
    rp = np.concatenate([[0], np.cumsum([len(c) for c in cols])]).astype(np.int64)
    csr = (n, m, rp, np.concatenate([np.asarray(c, np.int32) for c in cols]),
           (rng.random(int(rp[-1]), dtype=np.float32) - np.float32(0.5)))
    X = (rng.random((m, k), dtype=np.float32) - np.float32(0.5))
    X[m - 1] = np.inf  # column m - 1 has no entry
    with TiledMatrix(csr, **opts) as A:
        Y = A.spmm(torch.from_numpy(X).cuda()).cpu().numpy().astype(np.float64)
    for q in {0, k // 2, k - 1}:
        x = np.where(np.isinf(X[:, q]), np.float32(0), X[:, q])
        assert np.all(np.abs(Y[:, q] - oracle.spmv(csr, x)) <= TOL * oracle.absmv(csr, x)), q


@pytest.mark.parametrize("k", [2, 3, 7, 33])
def test_fused_restart_widths(k):
    from paper_1103_2405_amd import TiledMatrix
    g = gg.rmat(11, 8, seed=5)
    csr, seeds = gg.rwr_matrix(g), gg.rwr_seeds(g, k, 6)
    with TiledMatrix(csr, split_len=64) as W:
        R = W.rwr(seeds, 0.85, 0.0, 7)[0].cpu().numpy().astype(np.float64)
    ref, _, _ = oracle.rwr(csr, seeds, 0.85, 0.0, 7)
    assert np.abs(R - ref).sum(0).max() <= 1e-6
