"""The rule that says how many of a tile's columns the staged tile kernel holds
in LDS (host code, compiled here and called with made-up handles), on both sides
of each of its bounds."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

CU, LDS = 256, 40960
ROOM = LDS - 64
M3 = 3 << 20
BUF = 1 << 29  # floats of x that the buffer loads reach

# (lds_stage, n_cols, begin, end, nnz, hot_nnz, long, items) -> columns staged
CASES = [
    # a tile that fits: asked for, or 8 entries per float and compute unit
    ((1, 100, 0, 100, 1, 0, 1, 1), 100), ((0, 100, 0, 100, 1, 0, 1, 1), 0), ((-1, 100, 0, 100, 1, 0, 1, 1), 0),
    ((0, 100, 0, 100, 8 * 100 * CU, 0, 10 ** 6, 9), 100), ((0, 100, 0, 100, 8 * 100 * CU - 1, 0, 10 ** 6, 9), 0),
    ((1, 50000, 9000, 9000 + ROOM, 5, 0, 5, 9), ROOM), ((1, 50000, 9000, 9000 + LDS, 5, 0, 5, 9), ROOM),
    ((1, 50000, 9000, 9000 + LDS + 1, 5, 0, 5, 9), 0), ((-1, 100, 0, 100, 10 ** 9, 10 ** 9, 1, 9), 0),
    # a wider one, asked for or not: 3M entries, half of its columns' number in the staged ones, no long row
    ((0, 10 ** 6, 0, 10 ** 6, M3, 500000, 1536, 9), ROOM), ((1, 10 ** 6, 0, 10 ** 6, M3, 500000, 1536, 9), ROOM),
    ((-1, 10 ** 6, 0, 10 ** 6, M3, 500000, 1536, 9), 0), ((0, 10 ** 6, 0, 10 ** 6, M3 - 1, 500000, 1535, 9), 0),
    ((1, 10 ** 6, 0, 10 ** 6, M3 - 1, 500000, 1535, 9), 0), ((0, 10 ** 6, 0, 10 ** 6, M3, 499999, 1536, 9), 0),
    ((0, 10 ** 6, 0, 10 ** 6, M3, 500000, 1537, 9), 0), ((0, 10 ** 6, 5, 10 ** 6 + 5, 31 << 20, 10 ** 7, 15872, 9), ROOM),
    ((0, 3 * 10 ** 6, 10 ** 6, 2 * 10 ** 6, M3, 500000, 1536, 9), ROOM),  # the tile's width, not the matrix'
    ((0, 1000, 0, 1000, M3, M3, 1536, 9), 1000),  # one that fits, with few entries for its size
    # the buffer loads' reach, the item counter's, a device without the LDS
    ((0, BUF, 0, 10 ** 6, M3, 500000, 1536, 9), 0), ((0, BUF - 1, 0, 10 ** 6, M3, 500000, 1536, 9), ROOM),
    ((1, 100, 0, 100, 1, 0, 1, 2 ** 31), 0), ((1, 100, 0, 100, 1, 0, 1, 2 ** 31 - 1), 100)]


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    if not (os.path.exists(HIPCC) or shutil.which(HIPCC)):
        pytest.skip("no hipcc")
    exe = str(tmp_path_factory.mktemp("staging") / "staging")
    csrc = os.path.join(ROOT, "paper_1103_2405_amd", "csrc")
    subprocess.check_call([HIPCC, "-std=c++17", "-O1", "--offload-arch=gfx950", "--cuda-host-only", "-I", csrc, "-I",
                           os.path.join(ROOT, "include"), "-x", "hip", os.path.join(HERE, "tile_staging_main.cpp"),
                           os.path.join(csrc, "tc_mem.cpp"), "-o", exe], stderr=subprocess.DEVNULL)

    def call(cases, lds=LDS):
        text = "\n".join("%d %d %d %d %d %d %d %d %d %d" % (c[0], CU, lds, *c[1:]) for c in cases)
        return [int(v) for v in subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.split()]

    return call


def test_bounds(rule):
    assert rule([c for c, _ in CASES]) == [w for _, w in CASES]


def test_without_lds(rule):
    assert rule([c for c, _ in CASES], lds=0) == [0] * len(CASES)
