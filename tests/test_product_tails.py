"""Rows past the full rounds of a product's large tiles, which the same launch takes in tiles of 128 x 128 (gemm_tiles.h, gemm.hip)."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

import oracle
import test_gpu_small_products as products
from paper_2507_14959_amd import binding, synth
from test_product_tiles import CSRC, SHIM, TILES

MORE = """
extern "C" int large_rows(int rows, int N, int bm, int bn) { return large_tile_rows(rows, N, bm, bn); }
extern "C" long tail(int rows, int N) { return tail_tiles(rows, N); }
extern "C" int may(int bm, int bn, int mode, int ahead) { return has_tail(bm, bn, mode, ahead); }
extern "C" long run(int known, int rows, int N, int bm, int bn)          // workgroups of an XCD
{
    return xcd_workgroups((long)((rows + bm - 1) / bm) * ((N + bn - 1) / bn), true, known != 0, rows, N, bm, bn);
}
// The tile of workgroup 8 j + xcd of a launch whose true count is `rows`, as the kernel finds it: row, column, tile rows, tile columns
extern "C" int tile(int xcd, int j, int rows, int N, int bm, int bn, int *at)
{
    const int large = large_tile_rows(rows, N, bm, bn);
    int mt, tn;
    if (xcd_tile(xcd, j, (large + bm - 1) / bm, (N + bn - 1) / bn, panel_tiles(bn), mt, tn)) { at[0] = mt * bm; at[1] = tn * bn; at[2] = bm; at[3] = bn; return 1; }
    if (large < rows && xcd_tile(xcd, j, (rows - large + 127) / 128, (N + 127) / 128, panel_tiles(128), mt, tn)) {
        at[0] = large + mt * 128; at[1] = tn * 128; at[2] = at[3] = 128;
        return 1;
    }
    return 0;
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("tails")
    (d / "shim.cpp").write_text(SHIM + MORE)
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", f"-I{CSRC}", "-o", str(d / "shim.so"), str(d / "shim.cpp")], check=True)
    lib = ctypes.CDLL(str(d / "shim.so"))
    lib.pick.argtypes = [ctypes.c_int] * 6 + [ctypes.c_float] + [ctypes.c_int] * 3 + [ctypes.POINTER(ctypes.c_float)]
    lib.tail.restype = lib.run.restype = ctypes.c_long
    return lib


def workgroups(lib, xcd, j, rows, N, bm, bn):
    at = (ctypes.c_int * 4)()
    return tuple(at) if lib.tile(xcd, j, rows, N, bm, bn, at) else None


@pytest.mark.parametrize("bm,bn", [(256, 256), (256, 128)])
@pytest.mark.parametrize("N", [200, 768, 1032, 3072])
def test_every_row_is_taken_once_and_the_grid_is_large_enough(lib, bm, bn, N):
    tails = 0
    for rows in [*range(1, 30000, 971), 256 * 256, 256 * 256 + 1]:
        large = lib.large_rows(rows, N, bm, bn)
        n_tiles = -(-N // bn)
        assert large == rows or (large % bm == 0 and 0 < large < rows and lib.tail(rows - large, N) <= 256 and large // bm * n_tiles % 256 in (0, *range(257 - n_tiles, 256)))
        tails += large < rows
        run = lib.run(1, rows, N, bm, bn)
        for bound in (rows, rows + 971, 2 * rows):
            assert run <= lib.run(0, bound, N, bm, bn)           # (a launch whose count only the device knows)
        seen = np.zeros((rows // 128 + 2, n_tiles * bn // 128), dtype=int)
        for bid in range(8 * run):
            at = workgroups(lib, bid & 7, bid >> 3, rows, N, bm, bn)
            if at:
                seen[at[0] // 128:(at[0] + at[2]) // 128, at[1] // 128:(at[1] + at[3]) // 128] += 1
        assert np.all(seen[:-(-rows // 128), :-(-N // 128)] == 1)
        assert all(workgroups(lib, x, run, rows, N, bm, bn) is None for x in range(8))
    assert tails > 0


# blocks, tokens, contraction, columns, rank, branches: columns that fill no tile, blocks that reach from the large tiles into the small ones
CASES = [(334, 197, 768, 200, 16, 1), (252, 131, 768, 512, 8, 2), (168, 197, 768, 512, 8, 1),
         (334, 197, 768, 200, 4, 1), (168, 197, 768, 512, 4, 1)]       # ranks that are not fetched ahead


@pytest.mark.parametrize("case", CASES)
def test_the_sizes_below_have_a_tail(lib, case):
    n, T, K, N, r, per = case
    us = (ctypes.c_float * len(TILES))()
    assert TILES[lib.pick(n, T, K, N, r, 0, per, 1, 0, 1, us)] == "256x256", list(us)
    assert lib.large_rows(n * T, N, 256, 256) < n * T


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES)
def test_against_the_oracle(case):
    products.test_against_the_oracle(*case)


@pytest.mark.gpu
@pytest.mark.parametrize("D,Dm,hw,F,r", [
    (512, 512, 80, 165, 8),      # residual on 256 x 128, qkv and fc1 on 256 x 256
    (512, 1024, 112, 64, 16),
])
def test_layers_against_the_oracle(D, Dm, hw, F, r):
    cfg, w, frames, off, ids = synth.make_small_case(900 + hw, dtype=synth.DT_BF16, targets=15, L=2, F=F, r=r, max_set=2, n_adapters=5, D=D, heads=D // 64,
                                                     Dm=Dm, hw=hw, patch=8)
    got = binding.run_forward(binding.DeviceModel(cfg, w, L0=1), frames, off, ids)
    err = np.abs(got["logits"] - oracle.forward(cfg, w, frames, off, ids, L0=1)["logits"]).max()
    assert got["status"] == 0 and err < 8e-3                     # (as the layers of test_product_tiles.py)
