"""SpMM on one unsplit row of 2^31 - 64 entries, the longest that a matrix can
hold in whole steps of the row loop: its last step ends past 2^31."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def test_row_of_almost_2_31_entries():
    from paper_1103_2405_amd import DeviceCsr, TiledMatrix
    from paper_1103_2405_amd.tc import load_library
    if torch.cuda.mem_get_info()[0] < 80 << 30:
        pytest.skip("needs 80 GB of device memory")
    L, m = 2 ** 31 - 64, 1 << 16
    col = torch.arange(L, dtype=torch.int32, device="cuda").bitwise_and_(m - 1)
    val = torch.ones(L, device="cuda")
    x = (np.arange(m) % 7 - 3).astype(np.float32)
    want = int(x.sum()) * (L // m) + int(x[:L % m].sum())  # whole numbers below 2^24: exact
    csr = (1, m, torch.tensor([0, L], device="cuda"), col, val)
    with TiledMatrix(DeviceCsr(csr), split_len=0) as A:
        del csr, col, val
        Y = A.spmm(torch.from_numpy(x).cuda().reshape(m, 1))
        assert float(Y[0, 0]) == want
    torch.cuda.empty_cache()
    load_library().tc_release_cached_memory()
