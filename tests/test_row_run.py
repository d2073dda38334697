"""Where layers run as tiles that stay on their CUs (row_waves.h): the sizes of test_gpu_rowrun.py are among them, and the rule against the costs that it is made of."""
import ctypes
import subprocess

import pytest

import test_gpu_rowrun as sizes
from test_product_tiles import CSRC

SHIM = """
#include "row_waves.h"
extern "C" int faster(int T, int Dm, int r, int by_block, int F, int R)     // R < 0: F blocks, which the host knows
{
    return rowrun_faster(T, RR_D, Dm, r, by_block != 0, R < 0 ? known_count(F) : pair_count(F, R));
}
extern "C" float layer_us(int waves, int T, int r, int by_block, int blocks) { return row_layer_us(waves, T, r, by_block != 0, blocks); }
extern "C" int waves(int T, int Dm, int r, int by_block, int F) { return rowreg_waves(T, RR_D, Dm, r, by_block != 0, known_count(F)); }
"""


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    d = tmp_path_factory.mktemp("run")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", f"-I{CSRC}", "-o", str(d / "shim.so"), str(d / "shim.cpp")], check=True)
    lib = ctypes.CDLL(str(d / "shim.so"))
    lib.layer_us.restype = ctypes.c_float
    return lib


def _tasks(blocks, T):
    return blocks * ((T + 31) // 32)


@pytest.mark.parametrize("case", sizes.CASES)
def test_the_sizes_run_as_tiles(shim, case):
    T, F, Dm, r, targets, L, L0, per_frame, spare = case
    pairs = sum(1 + f % 8 % per_frame for f in range(F)) + spare
    if L0 > 0:
        assert shim.faster(T, Dm, 0, 0, F, -1) and _tasks(F, T) > 64
    if L0 < L:
        assert shim.faster(T, Dm, r, 1, F, pairs) and _tasks((F + pairs) // 2, T) > 64


# blocks known to the host: one round up to 256 tiles, two up to 512, never more
@pytest.mark.parametrize("T,r,blocks,taken", [(197, 8, 64, 1), (197, 0, 64, 1), (197, 0, 65, 0), (197, 8, 72, 1), (197, 8, 128, 1), (197, 8, 129, 0), (17, 8, 256, 1), (17, 0, 513, 0),
                                              (113, 0, 128, 1), (113, 8, 240, 1)])
def test_rounds(shim, T, r, blocks, taken):
    assert shim.faster(T, 768, r, int(r > 0), blocks, -1) == taken


def test_it_is_never_taken_where_two_launches_a_layer_cost_less(shim):
    for T in (5, 17, 50, 64, 65, 101, 113, 128, 129, 192, 193, 197, 224):
        for blocks in list(range(1, 140)) + [200, 256, 300, 512, 600]:
            for r in (0, 8):
                w = shim.waves(T, 768, r, int(r > 0), blocks)
                layer = shim.layer_us(w, T, r, int(r > 0), blocks) + 4.5 + blocks * T / 2700
                tiles = blocks * ((T + 63) // 64)
                want = tiles <= 512 and 26.5 * ((tiles + 255) // 256) < layer
                if abs(26.5 * ((tiles + 255) // 256) - layer) > 1e-3:
                    assert shim.faster(T, 768, r, int(r > 0), blocks, -1) == want
