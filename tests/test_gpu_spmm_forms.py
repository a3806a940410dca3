"""The forms of the SpMM kernel that the smaller tests do not reach: deep ones
(more than 2^18 columns; a row that one wavefront sums alone), and X past the
24-bit rows and the 2^31 bytes of the 32-bit addresses, on both sides of each
bound, against FP64 sums of the same entries."""
import pytest
import torch

pytestmark = pytest.mark.gpu

TOL = 1e-5  # of |A||x| per element: FP64 sums rounded once


def check(n, m, r, c, val, ks, **opts):
    from paper_1103_2405_amd import TiledMatrix, tc
    rp = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    rp[1:] = torch.cumsum(torch.bincount(r, minlength=n), 0)
    with TiledMatrix((n, m, rp, c.to(torch.int32), val), **opts) as A:
        for k in ks:
            X = torch.rand(m, k, device="cuda", generator=torch.Generator("cuda").manual_seed(k)) - 0.5
            Y = A.spmm(X, torch.full((n, k), float("nan"), device="cuda")).double()
            t = val.double()[:, None] * X[c].double()
            ref = torch.zeros(n, k, dtype=torch.float64, device="cuda").index_add_(0, r, t)
            bound = torch.zeros_like(ref).index_add_(0, r, t.abs())
            assert bool(((Y - ref).abs() <= TOL * bound).all()), k
            del X, Y
    torch.cuda.empty_cache()
    tc.load_library().tc_release_cached_memory()


def entries(n, m, nnz, seed, hub=0):
    """Sorted entries with skewed rows; the last column has some, row 1 has `hub` more."""
    g = torch.Generator("cuda").manual_seed(seed)
    r = (torch.rand(nnz, device="cuda", generator=g, dtype=torch.float64) ** 3 * n).long()
    c = torch.randint(0, m, (nnz,), device="cuda", generator=g)
    c[::97] = m - 1
    if hub:
        r = torch.cat([r, torch.ones(hub, dtype=torch.int64, device="cuda")])
        c = torch.cat([c, torch.randint(0, m, (hub,), device="cuda", generator=g)])
    key = torch.unique(r * m + c)
    return key // m, key % m, torch.rand(key.numel(), device="cuda", generator=g) - 0.5


@pytest.mark.parametrize("m", [1 << 18, (1 << 18) + 1])
@pytest.mark.parametrize("opts", [{}, dict(wl=96, split_len=64), dict(tile_width=100000, wl=512)])
def test_many_columns(m, opts):
    n = 3001
    check(n, m, *entries(n, m, 60000, 3), (16, 17, 32, 33, 40, 100), **opts)


@pytest.mark.parametrize("hub", [2047, 2048, 9001])
def test_unsplit_row(hub):
    n, m = 5003, 20011
    check(n, m, *entries(n, m, 30000, 5, hub), (1, 2, 3, 4, 5, 8, 9, 16, 17, 36), split_len=0)


@pytest.mark.parametrize("m,ks", [(1 << 24, (1, 2, 3, 4, 5, 8, 13, 17, 31)), ((1 << 24) + 1, (1, 2, 3, 4, 5, 8, 13, 17)),
                                  (1 << 24, (32,)), ((1 << 21) + 7, (255, 256))])
@pytest.mark.parametrize("opts", [dict(wl=128, split_len=64), dict(split_len=0)])
def test_large_x(m, ks, opts):
    n = 2003
    check(n, m, *entries(n, m, 20000, 7, 3000), ks, **opts)


@pytest.mark.parametrize("k", [2, 9, 32])
def test_large_x_restart(k):
    # the fused restart of the batched walk, past the 24-bit rows
    from paper_1103_2405_amd import TiledMatrix, tc
    n = (1 << 24) + 3
    i = torch.arange(n, device="cuda")
    rp = torch.arange(n + 1, device="cuda")
    with TiledMatrix((n, n, rp, ((i * 5 + 1) % n).to(torch.int32), torch.full((n,), 0.5, device="cuda"))) as W:
        seeds = [(n - 1 - 7 * q) for q in range(k)]
        R = W.rwr(seeds, 0.85, 0.0, 3)[0]
    got = torch.nonzero(R)
    c = float(torch.tensor(0.85))
    # r' = c W r + (1 - c) e: node j feeds the row i with 5 i + 1 = j (mod n)
    want = {}
    for q, s in enumerate(seeds):
        r = {s: 1.0}
        for _ in range(3):
            new = {s: 1.0 - c}
            for j, v in r.items():
                row = (j - 1) * pow(5, -1, n) % n
                new[row] = new.get(row, 0.0) + c * 0.5 * v
            r = new
        want.update({(a, q): v for a, v in r.items()})
    assert {tuple(v) for v in got.tolist()} == set(want)
    for (a, q), v in want.items():
        assert abs(float(R[a, q]) - v) <= 1e-6
    del R, W
    torch.cuda.empty_cache()
    tc.load_library().tc_release_cached_memory()
