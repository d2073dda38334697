"""Where layers run as tiles that stay on their CUs (row_waves.h): the sizes of test_gpu_rowrun.py are among them, and the rule against the costs that it is made of."""
import ctypes
import subprocess

import pytest

import test_gpu_rowrun as sizes
from test_product_tiles import CSRC

SHIM = """
#include "row_waves.h"
extern "C" int rows(int T, int Dm, int r, int by_block, int F, int R)     // R < 0: F blocks, which the host knows
{
    return rowrun_rows(T, RR_D, Dm, r, by_block != 0, R < 0 ? known_count(F) : pair_count(F, R));
}
extern "C" int rounds(int blocks, int tiles) { return rowrun_rounds(blocks, tiles); }
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
    rows, T, F, Dm, r, targets, L, L0, per_frame, spare = case
    pairs = sum(1 + f % 8 % per_frame for f in range(F)) + spare
    if L0 > 0:
        assert shim.rows(T, Dm, 0, 0, F, -1) in (32, 64) and _tasks(F, T) > 44
    if L0 < L:
        assert shim.rows(T, Dm, r, 1, F, pairs) == rows and _tasks((F + pairs) // 2, T) > 44


# blocks known to the host: one round of 32 rows, one of 64, two of either, never more than 512 tiles, or 1024 where the other way is tiles of 64 rows
@pytest.mark.parametrize("T,r,blocks,rows", [(197, 8, 36, 32), (197, 8, 37, 64), (197, 8, 64, 64), (197, 0, 64, 64), (197, 0, 65, 0), (197, 0, 85, 0), (197, 0, 86, 64), (197, 8, 64, 64), (197, 8, 72, 64), (197, 8, 128, 64),
                                             (197, 8, 129, 0), (17, 8, 256, 32), (17, 0, 513, 0), (113, 0, 64, 32), (113, 0, 128, 64), (113, 8, 240, 64), (17, 8, 513, 32), (17, 8, 1024, 32),
                                             (17, 8, 1025, 0)])
def test_rounds(shim, T, r, blocks, rows):
    assert shim.rows(T, 768, r, int(r > 0), blocks, -1) == rows


@pytest.mark.parametrize("tiles", range(1, 8))
def test_a_round_holds_whole_blocks(shim, tiles):
    """Queues of 32 CUs each: whole blocks at a time, but everything that fits at once starts at once."""
    for blocks in range(1, 300):
        want = 1 if blocks * tiles <= 256 else -(-blocks // (8 * (32 // tiles)))
        assert shim.rounds(blocks, tiles) == want


def test_it_is_never_taken_where_two_launches_a_layer_cost_less(shim):
    for T in (5, 17, 50, 64, 65, 101, 113, 128, 129, 192, 193, 197, 224):
        for blocks in list(range(1, 140)) + [200, 256, 300, 512, 600]:
            for r in (0, 8):
                layer = shim.layer_us(shim.waves(T, 768, r, int(r > 0), blocks), T, r, int(r > 0), blocks) + 4.5 + blocks * T / 2700 + (3 if T > 192 and blocks > 85 else 0)
                most = 512 if shim.waves(T, 768, r, int(r > 0), blocks) else 1024
                us = {}
                for rows, one in ((64, 24.5 + T / 100), (32, 18 + T / 80)):
                    tiles = -(-T // rows)
                    us[rows] = one * shim.rounds(blocks, tiles) if blocks * tiles <= most else 1e9
                best = min(us, key=us.get)
                if min(abs(layer - us[best]), abs(us[32] - us[64])) > 1e-3:
                    assert shim.rows(T, 768, r, int(r > 0), blocks, -1) == (best if us[best] < layer else 0)
