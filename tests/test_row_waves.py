"""Which row kernel a call takes (row_waves.h): the sizes of test_gpu_rowreg.py reach the kernels that their comments name."""
import ctypes
import subprocess

import pytest

import test_gpu_rowreg as sizes
from test_product_tiles import CSRC

SHIM = """
#include "row_waves.h"
extern "C" int waves(int T, int Dm, int r, int by_block, int F, int R)     // R < 0: F blocks, which the host knows
{
    return rowreg_waves(T, RR_D, Dm, r, by_block != 0, R < 0 ? known_count(F) : pair_count(F, R));
}
"""


@pytest.fixture(scope="module")
def waves(tmp_path_factory):
    d = tmp_path_factory.mktemp("waves")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", f"-I{CSRC}", "-o", str(d / "shim.so"), str(d / "shim.cpp")], check=True)
    return ctypes.CDLL(str(d / "shim.so")).waves


# waves of the shared layers and of the adapted ones, 0: tiles of 64 rows
WAVES = {(460, 768): (4, 4), (300, 128): (0, 4), (460, 192): (4, 4), (520, 320): (4, 4), (900, 256): (8, 8), (700, 192): (4, 0), (100, 768): (4, 4)}


@pytest.mark.parametrize("case", sizes.CASES)
def test_the_sizes_reach_the_kernels_they_are_for(waves, case):
    F, hw, patch, Dm, r, targets, per_frame, spare = case
    T, pairs = 1 + (hw // patch) ** 2, sum(1 + f % sizes.UNIQUE % per_frame for f in range(F))
    assert (waves(T, Dm, 0, 0, F, -1), waves(T, Dm, r, 1, F, pairs + spare)) == WAVES[F, Dm]


@pytest.mark.parametrize("F", sorted({F for F, _ in sizes.BOTH}))
def test_rows_past_full_rounds(waves, F):
    assert (waves(37, 128, 0, 0, F, -1), waves(37, 128, 8, 1, F, F)) == (12, 12) and waves(37, 128, 8, 1, F, F + 2) in (4, 8)
    assert waves(64, 768, 0, 0, 1024, -1) == 8 and waves(64, 768, 0, 0, 1025, -1) == 12 and waves(64, 768, 0, 0, 1537, -1) == 8


def test_the_lagged_loop_is_above_the_line(waves):
    F, hw, patch, Dm, r, room = sizes.LOOP
    assert waves(1 + (hw // patch) ** 2, Dm, 0, 0, F, -1) > 0 and waves(1 + (hw // patch) ** 2, Dm, r, 1, F, room * F) > 0


@pytest.mark.parametrize("F,spare,taken", sizes.ROOM)
def test_much_room_is_decided_at_one_adapter_a_frame(waves, F, spare, taken):
    assert (waves(37, 192, 8, 1, F, F), waves(37, 192, 8, 1, F, F + spare)) == (taken, taken)
    assert waves(37, 192, 8, 1, F + spare // 2, -1) > taken      # (half the room would say otherwise)
