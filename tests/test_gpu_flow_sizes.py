"""The task queue on both sides of its rules: proj in the tasks of the hidden layer or a step of its own, fine and coarse tasks."""
import numpy as np
import pytest

import oracle
from paper_2507_14959_amd import binding, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,Dm,hw,blocks,r,targets,L0,compose", [
    (192, 768, 32, 24, 8, 3, 1, "branch"),       # T = 17: 24 tiles, fine tasks with proj in F1
    (192, 768, 32, 25, 8, 3, 1, "branch"),       # 25: coarse ones
    (192, 768, 48, 12, 20, 15, 0, "branch"),     # T = 37, 24 tiles; two rank steps, the second of four; adapters on every linear
    (192, 768, 48, 32, 20, 15, 0, "branch"),     # 64
    (192, 768, 48, 33, 20, 15, 0, "branch"),     # 66: proj a step of its own
    (192, 768, 112, 3, 16, 2, 1, "branch"),      # T = 197, 21 tiles; adapters on proj only
    (192, 768, 112, 5, 16, 2, 1, "branch"),      # 35
    (192, 512, 80, 6, 8, 7, 0, "sum"),           # T = 101, 24 tiles; terms summed on proj
    (192, 512, 80, 16, 8, 7, 0, "sum"),          # 64
    (192, 512, 80, 17, 8, 7, 0, "sum"),          # 68
    (128, 384, 72, 10, 4, 10, 0, "branch"),      # T = 82, 30 tiles; a hidden width that coarse tasks do not divide
    (128, 384, 72, 11, 4, 10, 0, "sum"),         # 33
    (64, 256, 16, 64, 32, 15, 2, "branch"),      # T = 5; one column tile of proj a wave; the largest rank
])
def test_against_the_oracle(D, Dm, hw, blocks, r, targets, L0, compose):
    cfg, w, frames, _, _ = synth.make_small_case(940 + D + hw + r, dtype=synth.DT_BF16, targets=targets, L=3, F=blocks, r=r, n_adapters=5, D=D, heads=D // 64, Dm=Dm,
                                                 hw=hw, patch=8)
    rng = np.random.default_rng(blocks)
    off, ids = synth.sets_to_csr([np.sort(rng.choice(5, size=2 if compose == "sum" else 1, replace=False)) for _ in range(blocks)])
    model = binding.DeviceModel(cfg, w, L0=L0, compose=compose)
    got = binding.run_forward(model, frames, off, ids)
    again = binding.run_forward(model, frames, off, ids)
    want = oracle.forward(cfg, w, frames, off, ids, L0=L0, compose=compose)["logits"]
    err = np.abs(got["logits"] - want).max()
    print(f"logits max-abs error {err:.2e} of up to {np.abs(want).max():.2f}")
    assert got["status"] == 0 and np.array_equal(got["logits"], again["logits"])
    assert err < 8e-3


@pytest.mark.parametrize("dtype,D,bound", [(synth.DT_F32, 192, 2e-6), (synth.DT_BF16, 192, 8e-3), (synth.DT_BF16, 768, 8e-3)])
def test_keys_whose_scores_overflow_count_nothing(dtype, D, bound):
    """Every score of the second 32 keys is -infinity in 32 bits (-1e40), those of the first and the last key tile are not."""
    cfg, w, frames, _, _ = synth.make_small_case(880, dtype=dtype, targets=3, L=1, F=2, r=4, n_adapters=4, D=D, heads=D // 64, Dm=256, hw=64, patch=8)
    off, ids = synth.sets_to_csr([[0, 2], [3]])
    rng = np.random.default_rng(880)
    for n in ("patch_w", "patch_b", "cls", "ln1_b"):
        w[n] = np.zeros_like(w[n])
    d = rng.integers(1, 3, size=(cfg.T, D // 2)).astype(np.float32)
    keys = np.arange(cfg.T)
    d[(keys < 32) | (keys >= 64), 0] = 0                     # rows add up to nothing, so that a zero stays one when normalised
    w["pos"] = np.concatenate([d, -d], axis=1)
    w["qkv_w"][0, :, 0], w["qkv_b"][0, 0] = 0, 1e20          # first column of head 0's queries, and of its keys
    w["qkv_w"][0, :, D], w["qkv_b"][0, D] = 0, 0
    w["qkv_w"][0, 0, D] = -1e20
    got = binding.run_forward(binding.DeviceModel(cfg, w, L0=1), frames, off, ids)
    want = oracle.forward(cfg, w, frames, off, ids, L0=1)["logits"]
    assert got["status"] == 0 and np.abs(got["logits"][:len(ids)] - want).max() < bound
