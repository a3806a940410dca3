"""Products whose workloads are few and large: fewer of them than a workgroup of
the staged kernel has wavefronts, than the card has compute units, and one more;
the product in the caller's ids on both sides of the 1024 entries per workload up
to which it reads and writes through the maps.  The product in the caller's ids
has the bits of the one in internal ids, which is held to the oracle."""
import numpy as np
import pytest
import torch

import graphgen as gg
import oracle

pytestmark = pytest.mark.gpu

TOL = 1e-5  # of (|A||x|)_i: FP64 row sums rounded once


@pytest.mark.parametrize("wl", [1024, 1025, 8192])
@pytest.mark.parametrize("n_rows,n_cols,per", [(1000, 700, 9), (20011, 3001, 5), (20011, 300007, 13), (262144, 5003, 3),
                                               (262145, 5003, 3)])
@pytest.mark.parametrize("opts", [{}, dict(lds_stage=1), dict(slices=1), dict(slices=4)])
def test_product(n_rows, n_cols, per, wl, opts):
    from paper_1103_2405_amd import TiledMatrix
    rng = np.random.default_rng(n_rows + per)
    lens = rng.integers(0, 2 * per, n_rows)
    lens[:3] = (min(n_cols, 1500), 0, 300)
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    r = np.repeat(np.arange(n_rows), lens)
    c = (rng.integers(0, n_cols, n_rows)[r] + np.arange(r.size) - rp[r]) % n_cols
    order = np.lexsort((c, r))
    csr = (n_rows, n_cols, rp, c[order].astype(np.int32), gg.uniform_f32(r.size, 4))
    x = gg.uniform_f32(n_cols, 3)
    xd = torch.from_numpy(x).cuda()
    bound = TOL * oracle.absmv(csr, x)
    with TiledMatrix(csr, wl=wl, split_len=512, **opts) as A:
        y = A.spmv(xd, torch.full((n_rows,), float("nan"), device="cuda"))
        f = A.export_format()
        assert int(f["tile_wl"][0]) == wl
        assert np.all(np.abs(y.cpu().numpy().astype(np.float64) - oracle.spmv(csr, x)) <= bound)
        yi = torch.full((n_rows,), float("nan"), device="cuda")
        A.spmv_internal(xd[torch.from_numpy(f["cperm"].astype(np.int64)).cuda()], yi)
        assert torch.equal(yi[torch.from_numpy(f["rowmap"].astype(np.int64)).cuda()], y)
