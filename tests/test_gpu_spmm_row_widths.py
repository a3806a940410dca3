"""SpMM rows of the widths at which a row-major workload changes its loop (the
groups of a wavefront and twice as many, both sides), with workloads on both sides
of the 128 entries up to which a workload is cut into two row slices, and for every
way a wavefront divides into columns and groups, against FP64 sums."""
import pytest
import torch

pytestmark = pytest.mark.gpu

TOL = 1e-5  # of |A||x| per element: FP64 sums rounded once


@pytest.mark.parametrize("wl", [64, 128, 129, 300])
@pytest.mark.parametrize("per", [5, 8, 9, 16, 17, 31, 32, 33, 63, 64])
def test_rows(per, wl):
    from paper_1103_2405_amd import TiledMatrix
    n, m = 403, 1009
    g = torch.Generator("cuda").manual_seed(per)
    r = torch.arange(n, device="cuda").repeat_interleave(per)
    c = (torch.arange(n * per, device="cuda") * 31 + r) % m
    key = torch.unique(r * m + c)
    r, c = key // m, key % m
    val = torch.rand(key.numel(), device="cuda", generator=g) - 0.5
    rp = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    rp[1:] = torch.cumsum(torch.bincount(r, minlength=n), 0)
    with TiledMatrix((n, m, rp, c.to(torch.int32), val), wl=wl) as A:
        assert int(A.export_format(True)["tile_wl"][0]) == wl
        for k in (1, 2, 3, 4, 5, 7, 8, 13, 16, 23, 32, 37):
            X = torch.rand(m, k, device="cuda", generator=g) - 0.5
            Y = A.spmm(X, torch.full((n, k), float("nan"), device="cuda")).double()
            t = val.double()[:, None] * X[c].double()
            ref = torch.zeros(n, k, dtype=torch.float64, device="cuda").index_add_(0, r, t)
            bound = torch.zeros_like(ref).index_add_(0, r, t.abs())
            assert bool(((Y - ref).abs() <= TOL * bound).all()), k
