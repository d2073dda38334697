"""Products of the isolated linear: the few that run in one launch with the shrink, those whose contraction is split over the waves, and tiles that share a ring."""
import numpy as np
import pytest
import torch

import oracle
from paper_2507_14959_amd import binding, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_xblocks,T,K,N,r,per_block", [
    (1, 197, 768, 3072, 8, 1),       # 192 tiles of 64 x 64: one launch with the shrink
    (5, 197, 768, 768, 16, 2),       # 240: the same, two branches each
    (2, 131, 1088, 2048, 8, 1),      # 192
    (2, 131, 1088, 1600, 8, 1),      # 150
    (31, 17, 768, 1000, 20, 2),      # 272 tiles of 32 x 64: shared ring; a block ends inside nearly every tile; columns that fill no tile; two rank steps
    (28, 17, 768, 1000, 20, 2),      # 240: split contraction
    (31, 17, 1088, 1000, 8, 1),      # above a contraction of 1024, few enough tiles of 64 x 64: split contraction
    (64, 17, 1088, 1032, 8, 2),      # more of them: shared ring
    (4, 128, 512, 2112, 4, 1),       # the shortest contraction of the rule, whole row tiles
])
def test_against_the_oracle(n_xblocks, T, K, N, r, per_block):
    case = synth.make_lora_linear_case(dtype=synth.DT_BF16, seed=N + T, n_xblocks=n_xblocks, T=T, Kdim=K, Ndim=N, n_adapters=5, r=r, per_block=per_block)
    up = lambda a, dt=torch.bfloat16: torch.from_numpy(np.ascontiguousarray(a)).to(device="cuda", dtype=dt).contiguous()  # noqa: E731
    R = int(case["row_offsets"][-1])
    y = torch.full((R, T, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    ws = torch.empty(binding.poly_lora_linear_workspace_bytes(n_xblocks, T, r, R, synth.DT_BF16), dtype=torch.uint8, device="cuda")
    binding.poly_profile_begin(8)
    binding.poly_lora_linear(up(case["X"]), up(case["W"].T), up(case["bias"], torch.float32), up(np.swapaxes(case["A"], 1, 2)),
                             up(np.swapaxes(case["B"], 1, 2)), 0.75, up(case["row_offsets"], torch.int32), up(case["adapter_ids"], torch.int32), R, y, ws,
                             dev_status=status)
    torch.cuda.synchronize()
    prof = binding.poly_profile_end()
    one = n_xblocks * -(-T // 64) * -(-N // 64) <= 256 and n_xblocks + R <= 1024
    assert prof["shrink"]["launches"] == (0 if one else 1) and prof["gemm"]["launches"] == 1
    want = oracle.lora_linear(case, s=0.75)
    assert int(status.item()) == 0
    # bf16 (8 bits) rounds the output and every rank of the shrink output by at most 2^-8 of itself; sums are fp32
    slack = np.empty_like(want)
    for f in range(n_xblocks):
        for b in range(case["row_offsets"][f], case["row_offsets"][f + 1]):
            k = case["adapter_ids"][b]
            slack[b] = np.abs(0.75 * case["X"][f].astype(np.float64) @ case["A"][k]) @ np.abs(case["B"][k])
    over = np.abs(y.float().cpu().numpy() - want) - (2.0 ** -8 * np.abs(want) + 2.0 ** -8 * slack + 1e-4)
    assert over.max() <= 0


@pytest.mark.parametrize("n_xblocks,T,K,N,r,per_block", [
    (9, 197, 192, 576, 8, 2),        # two branches: the expand's operands fetched ahead
    (40, 37, 192, 200, 20, 3),       # 160 tiles of 64 x 64: one launch; blocks shorter than a wave's rows, columns that fill no tile, two rank steps
    (70, 37, 192, 200, 20, 3),       # 280: two
    (24, 131, 192, 1000, 8, 1),      # the last column tile cut short
    (30, 64, 320, 1032, 16, 2),      # as many rows as a taller wave's region: two blocks in it
])
def test_tiles_of_a_wave_per_32_rows(n_xblocks, T, K, N, r, per_block):
    test_against_the_oracle(n_xblocks, T, K, N, r, per_block)


@pytest.mark.parametrize("n_xblocks,T,K,N,r,per_block", [
    (30, 131, 64, 1032, 16, 2),      # one 64-column step: every load of the further stages is switched off
    (64, 197, 128, 768, 8, 1),       # as many steps as stages
    (100, 197, 192, 256, 20, 2),     # one more
])
def test_short_contractions(n_xblocks, T, K, N, r, per_block):
    test_against_the_oracle(n_xblocks, T, K, N, r, per_block)


@pytest.mark.parametrize("n_xblocks,T,K,N,r,per_block", [
    (128, 197, 768, 2304, 16, 1),    # tiles of 256 x 256
    (133, 197, 1536, 768, 16, 1),    # 128 x 128, a long contraction
])
def test_large_tiles(n_xblocks, T, K, N, r, per_block):
    test_against_the_oracle(n_xblocks, T, K, N, r, per_block)


@pytest.mark.parametrize("n_xblocks,T,K,N,r,per_block", [
    (60, 17, 192, 576, 4, 1),        # 64 x 64
    (256, 41, 192, 200, 20, 2),      # 128 x 128, column tiles cut short
    (256, 50, 192, 1032, 20, 1),
    (600, 101, 192, 200, 4, 1),      # a rank that fills no load
])
def test_ranks_that_are_not_fetched_ahead(n_xblocks, T, K, N, r, per_block):
    test_against_the_oracle(n_xblocks, T, K, N, r, per_block)
