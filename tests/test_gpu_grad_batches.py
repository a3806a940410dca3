"""The batches of the adjoint pass (whole checkpoint segments up to 32 steps, a
longer segment in pieces) and the rows of every entry, at the sizes where they
change: the gradient against FP64 and the same bits for every checkpoint
interval; the transpose's row ids with runs of empty rows."""
import numpy as np
import pytest
import torch

import graphgen as gg
from oracle import rwr_grad as rg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [1, 8, 9, 33, 40])
@pytest.mark.parametrize("opts", [{}, {"tile_width": 256}])  # one tile; several (the caller's ids)
def test_gradient_over_batches(K, opts):
    from paper_1103_2405_amd.rwr_grad import EdgeWeightedRWR
    g = gg.rmat(9, 24, seed=31)
    n, _, rp, col, _ = gg.rwr_matrix(g)
    feats = gg.normal_f32(len(col) * 3, 8).reshape(len(col), 3)
    seed = int(gg.rwr_seeds(g, 1, 2)[0])
    deg = np.diff(rp)
    targets = np.argsort(-deg)[:8].astype(np.int64)
    theta = np.array([0.3, -0.2, 0.5])
    targets = targets[targets != seed][:4] if K > 2 else np.array([seed])
    _, ref, _ = rg.loss_and_grad(n, rp, col, feats, theta, seed, targets, 0.85, K)
    got = []
    for every in (1, 5, 8, 50):
        model = EdgeWeightedRWR((n, n, rp, col), feats, seed, 0.85, K, every=every, build_opts=opts)
        th = torch.tensor(theta, dtype=torch.float64, requires_grad=True)
        (-torch.log(model.scores(th)[torch.from_numpy(targets).cuda()].double()).sum()).backward()
        got.append(th.grad.numpy().copy())
        model.close()
    for a in got:
        assert np.array_equal(a, got[0])
    # FP32 vectors: 1e-4 of the gradient, or of the sum's terms where it cancels (K = 1 from the seed itself)
    assert np.linalg.norm(got[0] - ref) <= 1e-4 * max(np.linalg.norm(ref), 1e-3)


@pytest.mark.parametrize("n_rows,lens", [(1, [5]), (3, [0, 1, 0]), (5000, "gaps"), (3, [0, 9001, 0]), (4097, "ones")])
def test_rows_of_entries(n_rows, lens):
    # the transpose carries each entry's row: blocks of 2,048 entries, empty rows
    # before, between and after, a row over several blocks
    import ctypes
    from paper_1103_2405_amd.tc import CCsr, load_library
    rng = np.random.default_rng(n_rows)
    if lens == "gaps":
        lens = np.where(np.arange(n_rows) % 1000 < 990, 0, rng.integers(0, 700, n_rows))
    elif lens == "ones":
        lens = np.ones(n_rows, np.int64)
    lens = np.asarray(lens, np.int64)
    rp = np.concatenate([[0], np.cumsum(lens)])
    nnz, m = int(rp[-1]), 9001
    col = np.concatenate([np.sort(rng.choice(m, int(k), replace=False)) for k in lens if k] or [np.zeros(0)]).astype(np.int32)
    d = [torch.from_numpy(a).cuda() for a in (rp, col, np.ones(nnz, np.float32))]
    rpT = torch.empty(m + 1, dtype=torch.int64, device="cuda")
    colT = torch.empty(nnz, dtype=torch.int32, device="cuda")
    A = CCsr(n_rows, m, nnz, d[0].data_ptr(), d[1].data_ptr(), d[2].data_ptr())
    vp = ctypes.c_void_p
    assert load_library().tc_csr_transpose(ctypes.byref(A), vp(rpT.data_ptr()), vp(colT.data_ptr()), vp(0), vp(0), vp(0)) == 0
    row = np.repeat(np.arange(n_rows), lens)
    order = np.argsort(col, kind="stable")
    assert np.array_equal(colT.cpu().numpy(), row[order].astype(np.int32))
    assert np.array_equal(rpT.cpu().numpy(), np.concatenate([[0], np.cumsum(np.bincount(col, minlength=m))]))
