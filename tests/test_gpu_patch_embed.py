"""The patch embedding: patches gathered by the product (patch.hip, gemm_ks.hip), and by a kernel of their own where the frames are not on a 16-byte boundary."""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2507_14959_amd import binding, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,F,H,W,patch,D,fused", [
    (synth.DT_F32, 3, 32, 32, 8, 128, True),        # 16 patches: half a tile
    (synth.DT_F32, 5, 24, 88, 8, 192, True),        # 33 patches of frames wider than high
    (synth.DT_F32, 1, 16, 16, 16, 128, True),       # one patch
    (synth.DT_F32, 40, 112, 64, 16, 192, True),     # 28 patches; tiles of 64
    (synth.DT_F32, 2, 32, 48, 4, 128, False),       # a contraction of 48: no whole number of k-tiles
    (synth.DT_F32, 2, 24, 24, 12, 128, False),      # .. and of 432
    (synth.DT_BF16, 1, 16, 16, 16, 64, True),       # one patch
    (synth.DT_BF16, 1, 224, 224, 16, 192, True),    # 196 patches: the last tile four rows
    (synth.DT_BF16, 4, 48, 240, 24, 128, True),     # 20 patches, a contraction of 1728
    (synth.DT_BF16, 7, 48, 64, 8, 192, True),       # 48 patches, three k-tiles: rows of a tile in three frames
    (synth.DT_BF16, 3, 224, 224, 16, 768, True),    # a wide model
    (synth.DT_BF16, 225, 224, 224, 16, 192, True),  # 2070 tiles of 64 x 64: those of 128 x 192, the last of 68 rows
    (synth.DT_BF16, 56, 224, 224, 16, 768, True),   # .. four of them side by side
    (synth.DT_BF16, 2, 24, 24, 12, 192, False),     # a run of 72 bytes: no whole number of pieces
])
def test_gathered_by_the_product_and_by_a_kernel(dtype, F, H, W, patch, D, fused):
    cfg, _, _, off, ids = synth.make_small_case(40 + F, dtype=dtype, F=F, L=1, n_adapters=4, D=D, heads=D // 64, hw=16, patch=8, targets=3, r=4)
    cfg = dataclasses.replace(cfg, H=H, W=W, patch=patch)
    rng = np.random.default_rng(F)
    model = binding.DeviceModel(cfg, synth.make_weights(cfg, rng), L0=0)
    frames = model.frames_to_device(synth.make_frames(cfg, F, rng))
    room = torch.empty(frames.numel() + 8, dtype=frames.dtype, device="cuda")
    assert frames.data_ptr() % 16 == 0 == room.data_ptr() % 16
    R = int(off[-1])
    o, i = (torch.from_numpy(a).to("cuda", torch.int32) for a in (off, ids))
    got, other = [], []
    for by in (0, 1):                                        # the same frames on a boundary and one element behind it
        room[by:by + frames.numel()] = frames.reshape(-1)
        ws = torch.full((binding.poly_forward_workspace_bytes(model, F, R),), 0xff, dtype=torch.uint8, device="cuda")
        scores, merged = torch.empty(R, cfg.C, device="cuda"), torch.empty(F, cfg.n_adapters, device="cuda")
        status = torch.full((1,), 99, dtype=torch.int32, device="cuda")
        binding.poly_profile_begin(400)
        try:
            binding.poly_forward(model, room[by:by + frames.numel()].view(frames.shape), o, i, R, scores, ws, out_merged=merged, dev_status=status)
        finally:
            prof = binding.poly_profile_end()
        assert status.item() == 0
        got.append((scores.cpu().numpy(), merged.cpu().numpy()))
        other.append(prof["other"]["launches"] if "other" in prof else 0)
    assert other[1] - other[0] == (1 if fused else 0)
    assert np.isfinite(got[0][0]).all()
    for a, b in zip(*got):
        if dtype == synth.DT_F32 or F > 7:
            np.testing.assert_array_equal(a, b)              # the same products of the same numbers in the same order
        else:
            # a short sum in one piece, or in four added up: fp32, sqrt(3072) 2^-24 = 3.3e-6 of embeddings of about one, which the first rounding to bf16 (2^-9) can
            # make a step of: scores, whose slope is 1/4 at most, differ by a step of the layer's bf16 values seen through one head
            np.testing.assert_allclose(a, b, rtol=0, atol=2 ** -9)
