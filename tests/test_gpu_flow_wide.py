"""The wide model's layers as tasks (flow_wide.hip), and layer by layer where the workspace has no room for the tasks."""
import numpy as np
import pytest
import torch

import oracle
from paper_2507_14959_amd import binding, synth
from test_gpu_workspace import _forward

pytestmark = pytest.mark.gpu


def _case(Dm, hw, r, targets, F, seed, L=2, max_set=2):
    return synth.make_small_case(seed, dtype=synth.DT_BF16, targets=targets, L=L, F=F, r=r, max_set=max_set, n_adapters=4, D=768, heads=12, Dm=Dm, hw=hw, patch=8)


@pytest.mark.parametrize("Dm,hw,r,targets,L0,F", [
    (3072, 112, 16, 15, 1, 1),       # T = 197: seven row tiles, the last of five rows; all twelve K steps of fc2 a wave
    (3072, 32, 8, 3, 0, 4),          # T = 17
    (256, 16, 4, 15, 0, 3),          # T = 5; the shortest contraction of fc2: a K step a wave
    (1536, 64, 12, 12, 2, 2),        # T = 65: a row in the last tile; no adapted layer
    (1280, 48, 16, 5, 1, 3),         # T = 37; ten steps of 32 a wave's last, adapters on qkv and fc1
])
def test_tasks_and_layer_by_layer_against_the_oracle(Dm, hw, r, targets, L0, F):
    cfg, w, frames, off, ids = _case(Dm, hw, r, targets, F, 860 + Dm + hw)
    model = binding.DeviceModel(cfg, w, L0=L0)
    want = oracle.forward(cfg, w, frames, off, ids, L0=L0)["logits"]
    full = torch.empty(binding.poly_forward_workspace_bytes(model, F, int(off[-1])), dtype=torch.uint8, device="cuda")
    err, size, first = {}, full.numel(), None
    while True:
        ws = full[:size]
        ws.fill_(0xff)                                       # nothing an earlier call left behind may be needed
        rc, got, status, prof = _forward(model, frames, off, ids, ws)
        if rc == binding.POLY_ECAP:
            break
        assert rc == 0 and status == 0
        n = prof["attention"]["launches"]
        err.setdefault(n, float(np.abs(got - want).max()))
        if n == 0:
            first = got if first is None else first
            assert np.array_equal(got, first)                # in one launch or several, run after run: the same bits
        size -= max(256, full.numel() // 24)
    print({k: f"{v:.2e}" for k, v in err.items()}, f"logits up to {np.abs(want).max():.2f}")
    assert 0 in err and max(err) >= cfg.L - L0
    assert max(err.values()) < 8e-3                          # (as the layers of test_product_tiles.py)


def test_rows_whose_mean_is_far_above_their_spread():
    """Rows of 20001 plus whole numbers that add up to nothing: the mean is exact, and so is the sum of a normalised row, whose elements come in pairs of one size.
    Values that sum it and a wide proj show a mean that is a rounding off (as in test_gpu_flow_fp32.py)."""
    cfg, w, frames, _, _ = _case(256, 32, 4, 3, 2, 890, L=1)
    off, ids = synth.sets_to_csr([[0], [1]])
    rng = np.random.default_rng(890)
    for n in ("patch_w", "patch_b", "cls", "qkv_b"):
        w[n] = np.zeros_like(w[n])
    d = rng.integers(-8, 9, size=(cfg.T, 384))
    w["pos"] = (20001 + np.concatenate([d, -d], axis=1)[:, rng.permutation(768)]).astype(np.float32)
    w["ln1_g"], w["ln1_b"] = np.ones_like(w["ln1_g"]), np.zeros_like(w["ln1_b"])
    w["qkv_w"][..., 1536:] = 1.0
    w["proj_w"] = synth.round_to_bf16(25 * w["proj_w"])
    binding.poly_profile_begin(100)
    try:
        got = binding.run_forward(binding.DeviceModel(cfg, w, L0=1), frames, off, ids)
    finally:
        prof = binding.poly_profile_end()
    err = np.abs(got["logits"] - oracle.forward(cfg, w, frames, off, ids, L0=1)["logits"]).max()
    print(f"{err:.2e}")
    # the stream is rounded to 2^-9 = 2e-3 of a spread of 5, 1.1e-4 rms; a head sums 768 of that times N(0, 0.02): 0.55 x 1.1e-4 twice, six of it at most.
    # 4e-2 with the mean a rounding off
    assert got["status"] == 0 and prof["attention"]["launches"] == 0 and err < 6e-4


@pytest.mark.parametrize("workgroups", [1, 3, 9])
def test_fewer_workgroups_than_queues_come_to_the_end(workgroups):
    """A workgroup that waits for what no running workgroup has drawn does it itself."""
    cfg, w, frames, off, ids = _case(512, 48, 8, 15, 2, 870)
    model = binding.DeviceModel(cfg, w, L0=1)
    all_of_them = binding.run_forward(model, frames, off, ids)
    binding.lib().poly_wait_workgroups(workgroups)
    try:
        few = binding.run_forward(model, frames, off, ids)
    finally:
        binding.lib().poly_wait_workgroups(0)
    assert few["status"] == 0 and all_of_them["status"] == 0 and np.array_equal(few["logits"], all_of_them["logits"])


def test_a_lone_workgroup_is_put_off_once_a_step_not_once_a_ticket():
    cfg, w, frames, off, ids = _case(512, 48, 8, 15, 2, 870)
    model = binding.DeviceModel(cfg, w, L0=0)
    want = binding.run_forward(model, frames, off, ids)
    tickets = len(ids) * 2 * (12 + 12 + 24 + 2 + 24)         # of a layer: two row tiles a block
    patience = 32 * 256                                      # put-offs of 256 looks each: more than the ten steps of two layers, less than the tickets of seven queues
    assert cfg.L == 2 and cfg.T == 37 and 10 < 32 < tickets * 7 // 8
    binding.lib().poly_wait_workgroups(1)
    binding.lib().poly_wait_limit(patience)
    try:
        alone = binding.run_forward(model, frames, off, ids)
    finally:
        binding.lib().poly_wait_workgroups(0)
        binding.lib().poly_wait_limit(-1)
    assert alone["status"] == 0 and np.array_equal(alone["logits"], want["logits"])


def test_no_patience_reports_a_stall_and_writes_no_row():
    cfg, w, frames, off, ids = _case(512, 48, 8, 15, 2, 871)
    model = binding.DeviceModel(cfg, w, L0=1)
    binding.lib().poly_wait_limit(0)
    try:
        got = binding.run_forward(model, frames, off, ids)
    finally:
        binding.lib().poly_wait_limit(-1)
    assert got["status"] == binding.POLY_ESTALL and np.isnan(got["logits"]).all()
    got = binding.run_forward(model, frames, off, ids)
    assert got["status"] == 0 and np.abs(got["logits"] - oracle.forward(cfg, w, frames, off, ids, L0=1)["logits"]).max() < 8e-3
