"""One-tile products that finish their split rows and write their rows without
entries in the tile's own launch, in internal and in the caller's ids: against
the oracle and the same bits call after call (the tickets of the split rows are
back at zero), on both sides of the sizes where the route changes."""
import numpy as np
import pytest
import torch

import graphgen as gg
import oracle

pytestmark = pytest.mark.gpu

TOL = 1e-5  # of (|A||x|)_i: FP64 row sums rounded once


def matrix(kind, n):
    if kind == "star":  # one row of many chunks (more than one round of 64 slots), most rows empty
        r, c = np.zeros(n, np.int64), np.arange(n)
    elif kind == "rows":  # three entries a row, none split, none empty
        r, c = np.repeat(np.arange(n), 3), (np.arange(3 * n) * 7919) % n
    else:
        return gg.pagerank_matrix(gg.rmat(int(np.log2(n)), 16, seed=9))
    key = np.unique(r * n + c)
    rp = np.zeros(n + 1, np.int64)
    np.add.at(rp, key // n + 1, 1)
    return n, n, np.cumsum(rp), (key % n).astype(np.int32), gg.uniform_f32(key.size, 4)


# up to 2^19 entries one launch through both maps, up to 2^18 rows rows through
# the map, above them two gathers
@pytest.mark.parametrize("kind,n,opts", [("star", 9000, dict(split_len=64)), ("star", 40000, dict()),
                                         ("rows", 1, dict()), ("rows", 65, dict(wl=64)), ("rows", 174762, dict()),
                                         ("rows", 174763, dict()), ("rows", 262144, dict()), ("rows", 262145, dict()),
                                         ("rmat", 1 << 14, dict(split_len=64)), ("rmat", 1 << 14, dict(relabel=0)),
                                         ("rmat", 1 << 16, dict(split_len=128, slices=4))])
def test_products(kind, n, opts):
    from paper_1103_2405_amd import TiledMatrix
    csr = matrix(kind, n)
    x = gg.uniform_f32(n, 3)
    xd = torch.from_numpy(x).cuda()
    bound = TOL * oracle.absmv(csr, x)
    ref = oracle.spmv(csr, x)
    with TiledMatrix(csr, **opts) as A:
        y = torch.full((n,), float("nan"), device="cuda")
        first = A.spmv(xd, y).clone()
        assert np.all(np.abs(first.cpu().numpy().astype(np.float64) - ref) <= bound)
        f = A.export_format(metadata_only=False)
        yi = torch.full((n,), float("nan"), device="cuda")
        A.spmv_internal(xd[torch.from_numpy(f["cperm"].astype(np.int64)).cuda()], yi)
        assert torch.equal(yi[torch.from_numpy(f["rowmap"].astype(np.int64)).cuda()], first)
        for _ in range(3):
            assert torch.equal(A.spmv(xd), first)


@pytest.mark.parametrize("n", [1 << 10, 1 << 14])
@pytest.mark.parametrize("panels", [0, -1])
def test_drivers_repeat(n, panels):
    # reductions finished in the launch that makes them: PageRank to a tolerance,
    # HITS and RWR give the same bits and the same change call after call
    from paper_1103_2405_amd import TiledMatrix
    g = gg.rmat(int(np.log2(n)), 8, seed=12)
    csr = gg.pagerank_matrix(g)
    with TiledMatrix(csr, panels=panels) as A:
        p, it, res = A.pagerank(0.85, 1e-6, 200, 5)
        q, jt, rs = A.pagerank(0.85, 0.0, it, 1)
        assert torch.equal(p, q) and it == jt and res == rs and 0 < res <= 1e-6
        ref, kt, _ = oracle.pagerank(csr, 0.85, 0.0, it)
        assert np.abs(p.cpu().numpy().astype(np.float64) - ref).sum() <= 1e-6
    with TiledMatrix(gg.hits_matrix(g), panels=panels) as B:
        a, h, it, res = B.hits(0.0, 9)
        b, k, _, rs = B.hits(0.0, 9)
        assert torch.equal(a, b) and torch.equal(h, k) and res == rs
