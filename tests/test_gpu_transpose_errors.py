"""tc_csr_transpose writes nothing for a matrix that it refuses, on both sides of
the sizes at which its column counts change; and the smallest it accepts."""
import ctypes

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def call(n, m, rp, col, rpT, colT, permT):
    from paper_1103_2405_amd.tc import CCsr, load_library
    d = [torch.from_numpy(np.asarray(rp, np.int64)).cuda(), torch.from_numpy(np.asarray(col, np.int32)).cuda()]
    vp = ctypes.c_void_p
    A = CCsr(n, m, len(col), d[0].data_ptr(), d[1].data_ptr(), None)
    st = load_library().tc_csr_transpose(ctypes.byref(A), vp(rpT.data_ptr()), vp(colT.data_ptr()), vp(0),
                                         vp(permT.data_ptr()), vp(0))
    torch.cuda.synchronize()
    return st


@pytest.mark.parametrize("nnz", [100, 4095, 4096, 70000])
@pytest.mark.parametrize("what", ["column", "order", "end"])
def test_refused_matrices_leave_the_outputs(nnz, what):
    from paper_1103_2405_amd import tc
    n, m = 50, 1000
    rp, col = np.linspace(0, nnz, n + 1).astype(np.int64), (np.arange(nnz) * 7) % m
    if what == "column":
        col[nnz // 2] = m
    elif what == "order":
        rp[20], rp[21] = rp[21], rp[20] - 1
    else:
        rp[n] = nnz - 1
    outs = [torch.full((k,), -77, dtype=t, device="cuda") for k, t in
            ((m + 1, torch.int64), (nnz, torch.int32), (nnz, torch.int32))]
    assert call(n, m, rp, col, *outs) == tc.TC_EINVAL
    assert all(bool((o == -77).all()) for o in outs)


@pytest.mark.parametrize("n,m,col", [(3, 0, []), (0, 3, []), (0, 0, []), (2, 1, [0, 0]), (1, 70001, [70000])])
def test_small_matrices(n, m, col):
    rp = np.zeros(n + 1, np.int64)
    if col:
        rp[-1] = len(col)
    outs = [torch.full((max(k, 1),), -77, dtype=t, device="cuda") for k, t in
            ((m + 1, torch.int64), (len(col), torch.int32), (len(col), torch.int32))]
    assert call(n, m, rp, col, *outs) == 0
    assert outs[0].tolist() == [0] * m + [len(col)] if not col or m > 1 else outs[0].tolist() == [0, len(col)]
    if col:
        assert outs[1].tolist() == [n - 1] * len(col) and outs[2].tolist() == list(range(len(col)))
