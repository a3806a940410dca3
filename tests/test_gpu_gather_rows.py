"""Rows gathered by an index list: every route (one float, four per thread; rows
of 16-byte pieces; any other width) around its remainders, from and to any
4-byte boundary.  Copies: bit equality."""
import ctypes

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("width", [1, 3, 4, 5, 8])
@pytest.mark.parametrize("n", [1, 3, 4, 5, 255, 1023, 1024, 1025, 100003])
@pytest.mark.parametrize("off", [(0, 0, 0), (1, 2, 3), (3, 1, 0)])
def test_gather(width, n, off):
    from paper_1103_2405_amd.tc import load_library
    g = torch.Generator(device="cuda")
    g.manual_seed(n + width)
    n_src = 777
    src = torch.rand(n_src * width + off[0], device="cuda", generator=g)[off[0]:]
    idx = torch.randint(0, n_src, (n + off[1],), dtype=torch.int32, device="cuda", generator=g)[off[1]:]
    buf = torch.full((n * width + off[2] + 1,), -1.0, device="cuda")
    dst = buf[off[2]:-1]
    vp = ctypes.c_void_p
    assert load_library().tc_gather_rows(vp(src.data_ptr()), n_src, vp(idx.data_ptr()), n, width,
                                         vp(dst.data_ptr()), None) == 0
    assert torch.equal(dst.view(n, width), src.view(n_src, width)[idx.long()])
    assert buf[-1] == -1.0 and torch.all(buf[:off[2]] == -1.0)
