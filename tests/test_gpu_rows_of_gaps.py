"""The row of every entry where blocks of 2,048 entries meet long runs of empty
rows (a block walks up to 32 x 256 rows, past that it searches each entry's
row), through the transpose and the coordinate build: whole numbers, exactly.
And no run of empty rows costs more than the matrix without it by much."""
import ctypes
import time

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

M = 5003


def matrix(n_rows, at, lens):
    """Rows `at` hold `lens` entries, the others none."""
    full = np.zeros(n_rows, np.int64)
    full[at] = lens
    rp = np.concatenate([[0], np.cumsum(full)])
    rng = np.random.default_rng(n_rows)
    col = np.concatenate([np.sort(rng.choice(M, int(k), replace=False)) for k in lens]).astype(np.int32)
    return rp, col


def transpose(n_rows, rp, col):
    from paper_1103_2405_amd.tc import CCsr, load_library
    d = [torch.from_numpy(a).cuda() for a in (rp, col, np.ones(col.size, np.float32))]
    rpT = torch.empty(M + 1, dtype=torch.int64, device="cuda")
    colT = torch.empty(col.size, dtype=torch.int32, device="cuda")
    vp = ctypes.c_void_p
    A = CCsr(n_rows, M, col.size, *(t.data_ptr() for t in d))

    def call():
        assert load_library().tc_csr_transpose(ctypes.byref(A), vp(rpT.data_ptr()), vp(colT.data_ptr()), vp(0), vp(0),
                                               vp(0)) == 0
        torch.cuda.synchronize()

    call()
    t = time.perf_counter()
    call()
    return colT.cpu().numpy(), time.perf_counter() - t


# rows of a block at, below and above the walk's 8,192; gaps before, inside and
# after a block's entries, gaps of one block only, every row after a gap
@pytest.mark.parametrize("n_rows,at,lens", [
    (8193, [0, 8192], [3, 5]), (8194, [0, 8193], [3, 5]), (8200, [0, 8190, 8191, 8192, 8193, 8194, 8199], [1] * 7),
    (100003, [0, 99999], [2047, 1]), (100003, [0, 99999], [2048, 1]), (100003, [50000, 100002], [2049, 4096]),
    (300007, [5, 9000, 18193, 27000, 200000, 300006], [700, 1, 1400, 5000, 4999, 13]),
    (2000003, list(range(100, 2000003, 1999)), [1 + q % 9 for q in range(len(range(100, 2000003, 1999)))])])
def test_rows(n_rows, at, lens):
    from paper_1103_2405_amd import TiledMatrix
    rp, col = matrix(n_rows, at, lens)
    row = np.repeat(np.arange(n_rows), np.diff(rp))
    colT, _ = transpose(n_rows, rp, col)
    assert np.array_equal(colT, row[np.argsort(col, kind="stable")].astype(np.int32))
    with TiledMatrix((n_rows, M, rp, col, np.ones(col.size, np.float32)), kernel="coo", relabel=0) as A:
        assert np.array_equal(A.export_format()["coo_row"], row.astype(np.int32))


def test_a_gap_costs_little():
    at, lens = [0, 1, (1 << 25) + 2], [2000, 3000, 4000]
    rp, col = matrix((1 << 25) + 3, at, lens)
    _, t = transpose((1 << 25) + 3, rp, col)
    # 2^25 rows walked by one block took 41 ms
    assert t < 10e-3
