"""Tiles wider than the staged columns with enough entries to be staged without
being asked for (3M and more): product, fused updates and the writers in the
caller's ids give the bits of the kernel that gathers every column through the
caches, and the oracle's bound holds; and matrices that the rule leaves to that
kernel (few entries in the hot columns, an unsplit hub row)."""
import numpy as np
import pytest
import torch

import graphgen as gg
import oracle

pytestmark = pytest.mark.gpu

TOL = 1e-5  # of (|A||x|)_i: FP64 row sums rounded once per tile


def skewed(n, nnz, power, hub, seed):
    """Square CSR, columns and a half of the rows skewed by `power`; hub: entries of row n // 2."""
    g = torch.Generator("cuda").manual_seed(seed)
    u = torch.rand(nnz, device="cuda", generator=g, dtype=torch.float64)
    r = torch.cat([torch.randint(0, n, (nnz // 2,), device="cuda", generator=g), (u[:nnz - nnz // 2] ** 6 * n).long()])
    c = (torch.rand(nnz, device="cuda", generator=g, dtype=torch.float64) ** power * n).long()
    if hub:
        r, c = torch.cat([r, torch.full((hub,), n // 2, device="cuda")]), torch.cat([c, torch.arange(hub, device="cuda")])
    key = torch.unique(r.clamp(max=n - 1) * n + c.clamp(max=n - 1))
    rp = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    rp[1:] = torch.cumsum(torch.bincount(key // n, minlength=n), 0)
    val = torch.rand(key.numel(), device="cuda", generator=g)
    return n, n, rp, (key % n).to(torch.int32), val


@pytest.mark.parametrize("n,nnz,power,hub,opts", [
    (40897, 7000000, 3, 0, {}), (65537, 7000000, 3, 0, dict(wl=96, slices=2)),
    (262145, 6000000, 3, 0, dict(slices=4)), (400001, 6000000, 3, 0, dict(tile_bounds=[5, 300000], slices=8)),
    (400001, 4200000, 2, 0, dict(wl=640, slices=1)), (1 << 19, 4200000, 4, 0, dict(tile_width=1 << 18)),
    # not staged: uniform columns past half their number, a hub row that one wavefront sums
    (1 << 20, 3600000, 1, 0, {}), (200001, 5000000, 3, 60000, dict(split_len=0))])
def test_staged_by_default(n, nnz, power, hub, opts):
    from paper_1103_2405_amd import DeviceCsr, TiledMatrix
    csr = skewed(n, nnz, power, hub, n)
    assert csr[3].numel() > 3 << 20
    A = DeviceCsr(csr)
    x = gg.uniform_f32(n + 1, 7)
    xd = torch.from_numpy(x).cuda()
    got = []
    for stage in (0, -1):
        with TiledMatrix(A, lds_stage=stage, **opts) as M:
            y = [torch.full((n,), float("nan"), device="cuda") for _ in range(2)]
            M.spmv_internal(xd[:n], y[0])
            M.spmv_internal(xd[1:], y[1])  # 4-byte aligned only
            got.append((M.spmv(xd[:n]), *y, M.pagerank(0.85, 0.0, 4)[0], M.rwr([n // 2], 0.85, 0.0, 4)[0]))
    for a, b in zip(*got):
        assert torch.equal(a, b)
    host = (n, n, csr[2].cpu().numpy(), csr[3].cpu().numpy(), csr[4].cpu().numpy())
    yh = got[0][0].cpu().numpy().astype(np.float64)
    assert np.all(np.abs(yh - oracle.spmv(host, x[:n])) <= TOL * oracle.absmv(host, x[:n]))
