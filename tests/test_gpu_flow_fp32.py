"""Single precision on few blocks: the layers as tasks (flow.hip) and, in a workspace without room for the tasks, layer by layer (gemm_ks.hip, attn_f32_kernel)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2507_14959_amd import binding, synth
from test_gpu_workspace import _forward

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,Dm,hw,r,targets,L0,compose", [
    (192, 768, 32, 4, 3, 0, "branch"),       # T = 17: every row tile cut short
    (192, 768, 112, 8, 15, 1, "branch"),     # T = 197: seven row tiles, the last of five rows; adapters on every linear
    (192, 384, 48, 20, 15, 0, "sum"),        # T = 37; two rank steps, the second of four; terms summed
    (192, 256, 16, 32, 15, 0, "branch"),     # T = 5; the largest rank
    (192, 640, 88, 12, 9, 2, "branch"),      # T = 122; no adapter on proj and fc1
    (192, 128, 48, 4, 15, 1, "sum"),         # the shortest contraction of fc2
    (192, 768, 88, 16, 5, 0, "branch"),      # 20 tiles and more of adapted blocks: tasks of twice the columns
])
def test_tasks_and_layer_by_layer_against_the_oracle(D, Dm, hw, r, targets, L0, compose):
    cfg, w, frames, off, ids = synth.make_small_case(830 + D + hw + r, dtype=synth.DT_F32, targets=targets, L=3, F=5, r=r, max_set=3, n_adapters=4, D=D,
                                                     heads=D // 64, Dm=Dm, hw=hw, patch=8)
    model = binding.DeviceModel(cfg, w, L0=L0, compose=compose)
    want = oracle.forward(cfg, w, frames, off, ids, L0=L0, compose=compose)["logits"]
    full = torch.empty(binding.poly_forward_workspace_bytes(model, 5, int(off[-1])), dtype=torch.uint8, device="cuda")
    err, size = {}, full.numel()
    while True:
        ws = full[:size]
        ws.fill_(0xff)                                       # nothing an earlier call left behind may be needed
        rc, got, status, prof = _forward(model, frames, off, ids, ws)
        if rc == binding.POLY_ECAP:
            break
        assert rc == 0 and status == 0
        err.setdefault(prof["attention"]["launches"], float(np.abs(got - want).max()))
        size -= max(256, full.numel() // 64)
    print({k: f"{v:.2e}" for k, v in err.items()}, f"logits up to {np.abs(want).max():.2f}")
    assert 0 in err and max(err) >= cfg.L - L0               # as tasks; layer by layer (the shared layers' tasks may find room still)
    # sums of up to 768 terms in another order than the oracle's: sqrt(768) 2^-24 = 1.7e-6 of values of about one, in every linear.  Measured up to 2e-7
    assert max(err.values()) < 2e-6


def test_rows_whose_mean_is_far_above_their_spread():
    """Rows of 1027 plus eighths that add up to nothing: their mean is exact, so a normalised row adds up to nothing but its own roundings, 2^-24 each.  Values
    that sum it and a wide proj show what more there is: a mean a rounding off, 2^-24 of 1027 in every element of the row, is 1e-3 and more in a logit."""
    cfg, w, frames, off, ids = synth.make_small_case(839, dtype=synth.DT_F32, targets=3, L=1, F=3, r=4, max_set=2, n_adapters=4, D=192, heads=3, Dm=384, hw=32, patch=8)
    rng = np.random.default_rng(839)
    for n in ("patch_w", "patch_b", "cls", "qkv_b"):
        w[n] = np.zeros_like(w[n])
    d = rng.integers(-12, 13, size=(cfg.T, 96)) / 8.0
    w["pos"] = (1027 + np.concatenate([d, -d], axis=1)[:, rng.permutation(192)]).astype(np.float32)
    w["ln1_g"], w["ln1_b"] = np.ones_like(w["ln1_g"]), np.zeros_like(w["ln1_b"])
    w["qkv_w"][..., 384:] = 1.0
    w["proj_w"] = (25 * w["proj_w"]).astype(np.float32)
    model = binding.DeviceModel(cfg, w, L0=1)
    want = oracle.forward(cfg, w, frames, off, ids, L0=1)["logits"]
    full = torch.empty(binding.poly_forward_workspace_bytes(model, 3, int(off[-1])), dtype=torch.uint8, device="cuda")
    rc, got, status, prof = _forward(model, frames, off, ids, full)
    err = np.abs(got - want).max()
    print(f"{err:.2e}", f"logits up to {np.abs(want).max():.2f}")
    assert rc == 0 and status == 0 and prof["attention"]["launches"] == 0
    # the stream itself is rounded to 2^-14 = 6e-5, twice; a head's sum of 192 such errors times N(0, 0.02): 0.28 x 3.5e-5 x 1.4 rms, six of it at most.  Measured 3.7e-5
    assert err < 8e-5
