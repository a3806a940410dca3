"""The builder's column counts, its first column without entries, its rows
without entries and its one-tile pack, at the edges of the counting kernels'
steps, slices, windows and of the rules between them: the column order is the
stable sort by decreasing length, whole numbers throughout, and products stay
within the FP64-sum bound."""
import numpy as np
import pytest
import torch

import graphgen as gg
import oracle

pytestmark = pytest.mark.gpu

TOL = 1e-5  # of (|A||x|)_i: FP64 row sums rounded once


def matrix(n_rows, n_cols, nnz, hub):
    # `hub` entries share column n_cols // 2, the others are spread; a quarter of
    # the rows stays empty, repeated entries are kept
    rng = np.random.RandomState(n_cols % 9973 + nnz)
    c = rng.randint(0, n_cols, nnz).astype(np.int64)
    c[rng.permutation(nnz)[:hub]] = n_cols // 2
    r = rng.randint(0, max(1, n_rows * 3 // 4), nnz).astype(np.int64)
    order = np.lexsort((c, r))
    rp = np.zeros(n_rows + 1, np.int64)
    np.add.at(rp, r + 1, 1)
    return n_rows, n_cols, np.cumsum(rp), c[order].astype(np.int32), gg.uniform_f32(nnz, 4)


CASES = [(300, 1, 5000, 0), (300, 4096, 4095, 0), (300, 4096, 4096, 0), (300, 4097, 8191, 100),
         (65536, 32768, 8193, 8193), (65537, 32769, (1 << 17) + 1, 70000), (131072, 40000, 1 << 18, 1 << 17),
         (131073, (1 << 20) + 1, 300001, 200000), (500, 1 << 25, 6000, 50), (500, (1 << 25) + 1, 6000, 50)]


@pytest.mark.parametrize("n_rows,n_cols,nnz,hub", CASES)
def test_counts(n_rows, n_cols, nnz, hub):
    from paper_1103_2405_amd import TiledMatrix
    csr = matrix(n_rows, n_cols, nnz, hub)
    clen = np.bincount(csr[3], minlength=n_cols)
    order = np.argsort(-clen, kind="stable")
    x = gg.uniform_f32(n_cols, 3)
    ref, bound = oracle.spmv(csr, x), TOL * oracle.absmv(csr, x)
    for opts in (dict(), dict(tile_width=1 << 20), dict(kernel="coo")):
        with TiledMatrix(csr, relabel=0, **opts) as A:
            assert np.array_equal(A.export_format()["cperm"], order)
            assert A.info()["n_dangling"] == np.count_nonzero(clen == 0)
            y = torch.full((n_rows,), float("nan"), device="cuda")
            A.spmv(torch.from_numpy(x).cuda(), y)
            assert np.all(np.abs(y.cpu().numpy().astype(np.float64) - ref) <= bound), opts


@pytest.mark.parametrize("nnz", [100, 5000])
@pytest.mark.parametrize("bad", [-1, 1000, 2**31 - 1, -2**31])
def test_ids_out_of_range_are_refused(nnz, bad):
    from paper_1103_2405_amd import TcError, TiledMatrix
    csr = matrix(300, 1000, nnz, 0)
    csr[3][nnz // 2] = bad
    with pytest.raises(TcError, match="column id"):
        TiledMatrix(csr)
