"""The last layer on the class token alone: every path behind attention, at the edges of the keys a lane group takes."""
import numpy as np
import pytest

import oracle
from paper_2507_14959_amd import synth
from test_gpu_forward import compare
from test_gpu_lora_linear import check, gpu_lora_linear

pytestmark = pytest.mark.gpu

BF, FP = synth.DT_BF16, synth.DT_F32


# patches of 8: 7 tokens or fewer keep all rows, 10 = fewer keys than lane groups, 65 and 145 one past the keys of 2 and 4 per group, 197 odd; fp32 122 and 226:
# a second and a third round of 112 keys
@pytest.mark.parametrize("dtype,D,heads,Dm,h,w_,r,targets,L,L0", [
    (BF, 512, 8, 512, 16, 24, 8, 15, 1, 0),          # 7 tokens
    (BF, 512, 8, 512, 24, 24, 20, 15, 1, 0),         # the only layer fans out; GEMM path
    (BF, 512, 8, 512, 64, 64, 16, 15, 2, 1),
    (BF, 512, 8, 512, 96, 96, 16, 5, 2, 2),          # no adapted layer
    (BF, 768, 12, 512, 112, 112, 16, 15, 2, 0),
    (BF, 192, 3, 384, 64, 64, 8, 15, 2, 1),          # tasks
    (FP, 64, 1, 128, 88, 88, 4, 15, 2, 1),
    (FP, 64, 1, 128, 120, 120, 6, 3, 1, 0),
    (FP, 192, 3, 256, 64, 72, 4, 3, 2, 2),
])
@pytest.mark.parametrize("compose", ["branch", "sum"])
def test_against_the_oracle(dtype, D, heads, Dm, h, w_, r, targets, L, L0, compose):
    from dataclasses import replace
    cfg, _, _, off, ids = synth.make_small_case(600 + D + h + L0, dtype=dtype, targets=targets, L=L, F=7, r=r, max_set=3, n_adapters=5, D=D, heads=heads, Dm=Dm, hw=16, patch=8)
    cfg = replace(cfg, H=h, W=w_)
    rng = np.random.default_rng(h + w_)
    compare(cfg, synth.make_weights(cfg, rng), synth.make_frames(cfg, 7, rng), off, ids, L0, K=cfg.n_adapters * cfg.C, compose=compose, tol=8e-3 if dtype == BF else None)


# the row kernels behind attention: more blocks than run as tasks (140 tiles of 32 rows), in tiles of 64 class rows with and without adapters
@pytest.mark.parametrize("targets,L0,r", [(3, 0, 8), (1, 1, 16), (3, 2, 8)])
def test_row_kernels_against_the_oracle(targets, L0, r):
    cfg, w, frames, off, ids = synth.make_small_case(71 + targets + L0, dtype=BF, targets=targets, L=2, F=75, r=r, max_set=2, n_adapters=5, D=192, heads=3, Dm=384, hw=56, patch=8)
    compare(cfg, w, frames, off, ids, L0, K=cfg.n_adapters * cfg.C, tol=8e-3)


# blocks of one row with a low-rank term each
@pytest.mark.parametrize("shape", [
    dict(n_xblocks=70, T=1, Kdim=192, Ndim=576, n_adapters=6, r=8, per_block=2),
    dict(n_xblocks=33, T=1, Kdim=768, Ndim=200, n_adapters=3, r=20, per_block=1),
])
def test_linear_on_blocks_of_one_row(shape):
    case = synth.make_lora_linear_case(dtype=BF, seed=77, **shape)
    Y, st = gpu_lora_linear(case, scale=1.5)
    assert st == 0
    check(Y, oracle.lora_linear(case, s=1.5), BF)


# many of them, on either side of where the split contraction is faster (ranks above 16, one round of 64 x 64 tiles, or two); all above the calls that are one launch
@pytest.mark.parametrize("shape", [
    dict(n_xblocks=2500, T=1, Kdim=192, Ndim=576, n_adapters=6, r=8, per_block=2),
    dict(n_xblocks=700, T=1, Kdim=192, Ndim=200, n_adapters=6, r=40, per_block=2),
    dict(n_xblocks=1100, T=1, Kdim=768, Ndim=1032, n_adapters=3, r=20, per_block=1),
    dict(n_xblocks=2300, T=1, Kdim=192, Ndim=760, n_adapters=6, r=36, per_block=1),
])
def test_linear_on_many_blocks_of_one_row(shape):
    case = synth.make_lora_linear_case(dtype=BF, seed=79, **shape)
    Y, st = gpu_lora_linear(case, scale=1.5)
    want = oracle.lora_linear(case, s=1.5)
    # the shrink output, scaled, and the result are rounded to eight bits, 2^-8 of them at most each; sums are in fp32
    frame = np.repeat(np.arange(shape["n_xblocks"]), np.diff(case["row_offsets"]))
    low = np.abs(1.5 * np.einsum("rk,rkq->rq", case["X"][frame, 0].astype(np.float64), case["A"][case["adapter_ids"]].astype(np.float64)))
    bound = 2.0 ** -8 * (np.abs(want[:, 0]) + np.einsum("rq,rqn->rn", low, np.abs(case["B"][case["adapter_ids"]]))) * 1.01 + 2e-5
    assert st == 0 and (np.abs(Y - want)[:, 0] <= bound).all(), (np.abs(Y - want)[:, 0] / bound).max()
