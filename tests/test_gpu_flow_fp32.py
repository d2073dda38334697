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
