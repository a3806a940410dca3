"""Many-graph RWR where many graphs' workloads begin within one step of the
segment table, where one graph spans many steps, and where graphs have no
workload at all: every graph's scores are those of the single-graph driver."""
import numpy as np
import pytest
import torch

import graphgen as gg

pytestmark = pytest.mark.gpu


def star(n):  # node 0 linked with every other node, both ways, columns of sum 1
    r = np.concatenate([np.zeros(n - 1, np.int64), np.arange(1, n)])
    c = np.concatenate([np.arange(1, n), np.zeros(n - 1, np.int64)])
    rp = np.zeros(n + 1, np.int64)
    np.add.at(rp, r + 1, 1)
    v = np.where(c == 0, 1.0 / max(n - 1, 1), 1.0).astype(np.float32)
    return n, n, np.cumsum(rp), c.astype(np.int32), v


def empty(n):
    return n, n, np.zeros(n + 1, np.int64), np.zeros(0, np.int32), np.zeros(0, np.float32)


@pytest.mark.parametrize("iters", [1, 8])
@pytest.mark.parametrize("width", [0, 64])  # one tile, several tiles
def test_many_segments(iters, width):
    from paper_1103_2405_amd import TiledMatrix, rwr_multi
    csrs = [star(2 + k % 90) for k in range(150)]
    csrs.insert(60, gg.rwr_matrix(gg.rmat(13, 16, seed=3)))
    csrs.insert(61, empty(5))
    csrs.append(empty(1))
    mats = [TiledMatrix(c, tile_width=width) for c in csrs]
    seeds = [c[0] // 2 for c in csrs]
    out, it, _ = rwr_multi(mats, seeds, 0.85, 0.0, iters, 1, graph=False)
    assert it == iters
    for m, s, r in zip(mats, seeds, out):
        assert torch.equal(m.rwr([s], 0.85, 0.0, iters)[0][:, 0], r)
