"""SpMM around the widths where tc_spmm pads the rows of its copy of X, on a
rectangle and on a relabelled square matrix, against FP64 sums."""
import numpy as np
import pytest
import torch

import graphgen as gg
import oracle

pytestmark = pytest.mark.gpu

TOL = 1e-5  # of (|A||X|)_ij: FP64 row sums rounded once a tile


@pytest.mark.parametrize("k", [4, 5, 8, 9, 12, 16, 17, 18, 19, 31, 32, 33, 36, 63, 255])
@pytest.mark.parametrize("kind", ["rectangle", "rmat"])
def test_widths(k, kind):
    from paper_1103_2405_amd import TiledMatrix
    if kind == "rmat":
        csr = gg.pagerank_matrix(gg.rmat(10, 8, seed=5))
    else:
        rng = np.random.RandomState(k)
        n_rows, n_cols, nnz = 333, 1001, 9000
        r = np.sort(rng.randint(0, n_rows, nnz))
        rp = np.zeros(n_rows + 1, np.int64)
        np.add.at(rp, r + 1, 1)
        csr = (n_rows, n_cols, np.cumsum(rp), rng.randint(0, n_cols, nnz).astype(np.int32), gg.uniform_f32(nnz, 4))
    X = gg.uniform_f32(csr[1] * k, 7).reshape(csr[1], k)
    with TiledMatrix(csr, relabel=1 if kind == "rmat" else 0) as A:
        Y = torch.full((csr[0], k), float("nan"), device="cuda")
        A.spmm(torch.from_numpy(X).cuda(), Y)
        got = Y.cpu().numpy().astype(np.float64)
    for c in {0, k // 2, k - 1}:
        x = np.ascontiguousarray(X[:, c])
        assert np.all(np.abs(got[:, c] - oracle.spmv(csr, x)) <= TOL * oracle.absmv(csr, x)), c
