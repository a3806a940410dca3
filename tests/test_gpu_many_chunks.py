"""One-tile formats with as many chunks as their products finish in the tile's own
launch (5,632) and with more, which a launch after it finishes: the product in
internal and in the caller's ids and the fused updates against the oracle, the
same bits call after call and under both tile kernels."""
import numpy as np
import pytest
import torch

import graphgen as gg
import oracle

pytestmark = pytest.mark.gpu

TOL = 1e-5  # of (|A||x|)_i: FP64 row sums rounded once


def matrix(n, lens):
    rng = np.random.default_rng(len(lens))
    at = np.sort(rng.choice(n, len(lens), replace=False))
    full = rng.integers(0, 3, n)
    full[at] = lens
    rp = np.concatenate([[0], np.cumsum(full)]).astype(np.int64)
    start = rng.integers(0, n, n)  # a row's columns: consecutive ones from a random start
    r = np.repeat(np.arange(n), full)
    c = (start[r] + np.arange(r.size) - rp[r]) % n
    order = np.lexsort((c, r))
    return n, n, rp, c[order].astype(np.int32), gg.uniform_f32(r.size, 4) / np.float32(64)


@pytest.mark.parametrize("lens,chunks", [([128] * 2816, 5632), ([128] * 2815 + [129], 5633), ([65] * 5000, 10000),
                                         ([20000, 9000] + [70] * 2600, 5654)])
@pytest.mark.parametrize("n,opts", [(30000, {}), (300000, {}), (30000, dict(lds_stage=1)), (30000, dict(slices=4, wl=512))])
def test_products_and_updates(n, opts, lens, chunks):
    from paper_1103_2405_amd import TiledMatrix
    csr = matrix(n, lens)
    x = gg.uniform_f32(n, 3)
    xd = torch.from_numpy(x).cuda()
    ref, bound = oracle.spmv(csr, x), TOL * oracle.absmv(csr, x)
    with TiledMatrix(csr, split_len=64, **opts) as A:
        assert A.info()["n_partials"] == chunks
        first = A.spmv(xd, torch.full((n,), float("nan"), device="cuda")).clone()
        assert np.all(np.abs(first.cpu().numpy().astype(np.float64) - ref) <= bound)
        f = A.export_format()
        yi = torch.full((n,), float("nan"), device="cuda")
        A.spmv_internal(xd[torch.from_numpy(f["cperm"].astype(np.int64)).cuda()], yi)
        assert torch.equal(yi[torch.from_numpy(f["rowmap"].astype(np.int64)).cuda()], first)
        assert torch.equal(A.spmv(xd), first)
        seeds = [int(np.argmax(np.diff(csr[2]))), 7]
        one = [A.rwr([s], 0.85, 0.0, 5)[0][:, 0] for s in seeds]
        both = A.rwr(seeds, 0.85, 0.0, 5)[0]
        want, _, _ = oracle.rwr(csr, np.array(seeds, np.int32), 0.85, 0.0, 5)
        for q in range(2):
            assert np.all(np.abs(one[q].cpu().numpy() - want[:, q]) <= 1e-5 * np.abs(want[:, q]) + 1e-7)
            assert np.all(np.abs(both[:, q].cpu().numpy() - want[:, q]) <= 1e-5 * np.abs(want[:, q]) + 1e-7)
        p = A.pagerank(0.85, 0.0, 5)[0]
        assert torch.equal(p, A.pagerank(0.85, 0.0, 5)[0])
        want, _, _ = oracle.pagerank(csr, 0.85, 0.0, 5)
        assert np.all(np.abs(p.cpu().numpy() - want) <= 1e-5 * np.abs(want) + 1e-9)
