"""Scratch of the adjoint pass: within what its interface states for every
checkpoint interval, in batches that the budget cuts, and the smallest form
where the device has not the memory; the same bits each time."""
import ctypes

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

vp = ctypes.c_void_p


def parts(n, every, K, opts):
    """A ring with chords, its handles, transposed structure and checkpoints."""
    from paper_1103_2405_amd.rwr_grad import EdgeWeightedRWR
    i = torch.arange(n, device="cuda")
    col = torch.stack([(i + 1) % n, (i * 7 + 3) % n], 1).sort(1)[0].flatten().to(torch.int32)
    rp = 2 * torch.arange(n + 1, device="cuda")
    feats = torch.linspace(-1, 1, 2 * n, device="cuda").view(2 * n, 1)
    m = EdgeWeightedRWR((n, n, rp, col), feats, 5, 0.85, K, every=every, build_opts=opts)
    m.forward(np.array([0.4]))
    return m


def adjoint(m, gK, G, g0):
    from paper_1103_2405_amd.rwr_grad import _ptr
    from paper_1103_2405_amd.tc import _check, _stream, load_library
    G.fill_(float("nan"))
    _check(load_library().tc_rwr_adjoint(m.W.handle, m.Wt.handle, _ptr(m.rpT), _ptr(m.colT), m.seed, m.c, m.K, m.every,
                                         _ptr(m.ckpt), _ptr(gK), _ptr(G), _ptr(g0), _stream()), "tc_rwr_adjoint")
    torch.cuda.synchronize()


def taken(f):
    from paper_1103_2405_amd.tc import load_library
    torch.cuda.synchronize()
    load_library().tc_release_cached_memory()
    a = torch.cuda.mem_get_info()[0]
    f()
    return a - torch.cuda.mem_get_info()[0]  # the pool keeps what the call took


@pytest.mark.parametrize("n,K,opts,everys", [(1 << 22, 12, {}, (1, 9, 12)), (1 << 23, 10, {}, (1, 9)),
                                             (1 << 22, 10, {"tile_width": 1 << 20}, (1, 9))])
def test_scratch_bound(n, K, opts, everys):
    first = None
    gK = torch.rand(n, device="cuda", generator=torch.Generator("cuda").manual_seed(3))
    G, g0 = torch.empty(2 * n, dtype=torch.float64, device="cuda"), torch.empty(n, device="cuda")
    for every in everys:
        m = parts(n, every, K, opts)
        used = taken(lambda: adjoint(m, gK, G, g0))
        vec, few = 4 * n, 8 if opts else 2  # several tiles: also split rows' sums and the like
        assert used <= max(1 << 30, (2 * every + 17) * vec) + 4 * 2 * n + (few + 2) * vec, (every, used)
        if first is None:
            first = G.clone(), g0.clone()
        assert torch.equal(G, first[0]) and torch.equal(g0, first[1])
        m.close()


@pytest.mark.parametrize("opts", [{}, {"tile_width": 1 << 20}])
def test_little_memory(opts):
    from paper_1103_2405_amd.tc import load_library
    n, K = 1 << 22, 12
    gK = torch.rand(n, device="cuda", generator=torch.Generator("cuda").manual_seed(3))
    G, g0 = torch.empty(2 * n, dtype=torch.float64, device="cuda"), torch.empty(n, device="cuda")
    m = parts(n, 5, K, opts)
    adjoint(m, gK, G, g0)
    want = G.clone(), g0.clone()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    load_library().tc_release_cached_memory()
    # room for the 2 x 5 + 1 vectors (184 MB) and the row ids, not for 2 x 5 + 17
    left = (2 * 5 + 1 + (2 if opts else 0) + 6) * 4 * n + 4 * 2 * n
    big = torch.empty(torch.cuda.mem_get_info()[0] - (2 << 30), dtype=torch.uint8, device="cuda")
    small = []
    try:
        while len(small) < 1024:
            small.append(torch.empty(32 << 20, dtype=torch.uint8, device="cuda"))
    except torch.OutOfMemoryError:
        pass
    del small[:-(-left // (32 << 20))]
    torch.cuda.empty_cache()
    try:
        adjoint(m, gK, G, g0)
    finally:
        del big, small
        torch.cuda.empty_cache()
        load_library().tc_release_cached_memory()
    assert torch.equal(G, want[0]) and torch.equal(g0, want[1])
    m.close()
