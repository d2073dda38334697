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
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("tails")
    (d / "shim.cpp").write_text(SHIM + MORE)
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", f"-I{CSRC}", "-o", str(d / "shim.so"), str(d / "shim.cpp")], check=True)
    lib = ctypes.CDLL(str(d / "shim.so"))
    lib.pick.argtypes = [ctypes.c_int] * 6 + [ctypes.c_float] + [ctypes.c_int] * 3 + [ctypes.POINTER(ctypes.c_float)]
    lib.tail.restype = ctypes.c_long
    return lib


def workgroups(xcd, j, rows, N, bm, bn, large):
    """The tile that workgroup 8 j + xcd takes, as the kernel finds it: (row, column, tile rows, tile columns), or None."""
    for m_tiles, n_tiles, row0, hm, hn in ((-(-large // bm), -(-N // bn), 0, bm, bn), (-(-(rows - large) // 128), -(-N // 128), large, 128, 128)):
        panel, total = 768 // hn, m_tiles * n_tiles
        lo, hi = total * xcd // 8, total * (xcd + 1) // 8
        if lo + j >= hi:
            j -= hi - lo
            continue
        pn, rem = divmod(lo + j, m_tiles * panel)
        width = min(panel, n_tiles - pn * panel)
        return row0 + rem // width * hm, (pn * panel + rem % width) * hn, hm, hn
    return None


@pytest.mark.parametrize("bm,bn", [(256, 256), (256, 128)])
@pytest.mark.parametrize("N", [200, 768, 1032, 3072])
def test_every_row_is_taken_once_and_the_grid_is_large_enough(lib, bm, bn, N):
    tails = 0
    for rows in [*range(1, 30000, 971), 256 * 256, 256 * 256 + 1]:
        large = lib.large_rows(rows, N, bm, bn)
        n_tiles = -(-N // bn)
        assert large == rows or (large % bm == 0 and 0 < large < rows and lib.tail(rows - large, N) <= 256 and large // bm * n_tiles % 256 in (0, *range(257 - n_tiles, 256)))
        tails += large < rows
        run = -(-(-(-large // bm) * n_tiles) // 8) + -(-lib.tail(rows - large, N) // 8)
        bound = -(-(-(-rows // bm) * n_tiles) // 8) + 32
        assert run <= bound                                      # (a launch whose count only the device knows)
        seen = np.zeros((rows // 128 + 2, n_tiles * bn // 128), dtype=int)
        for bid in range(8 * run):
            at = workgroups(bid & 7, bid >> 3, rows, N, bm, bn, large)
            if at:
                seen[at[0] // 128:(at[0] + at[2]) // 128, at[1] // 128:(at[1] + at[3]) // 128] += 1
        assert np.all(seen[:-(-rows // 128), :-(-N // 128)] == 1)
        assert all(workgroups(x, run, rows, N, bm, bn, large) is None for x in range(8))
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
