"""The kernels that go layer by layer on narrow bf16 models.

A call on few blocks runs its layers as tasks (flow.hip) when the workspace has room for the tasks' buffers, so these calls either have
many blocks or the smallest workspace the library takes.  Every test checks that attention was launched once per layer: what ran were the
row kernels (rowlayer.hip, rowlin.hip), the feed-forward kernel (mlp.hip) or the GEMM path.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2507_14959_amd import binding, synth

pytestmark = pytest.mark.gpu

TOL = 2e-2


class Call:
    def __init__(self, cfg, w, frames, off, ids, L0, compose="branch"):
        dev = "cuda"
        self.cfg, self.R = cfg, int(off[-1])
        self.model = binding.DeviceModel(cfg, w, L0=L0, compose=compose)
        self.frames = self.model.frames_to_device(frames)
        self.off, self.ids = torch.from_numpy(off).to(dev, torch.int32), torch.from_numpy(ids).to(dev, torch.int32)
        self.ws = torch.empty(binding.poly_forward_workspace_bytes(self.model, len(frames), self.R), dtype=torch.uint8, device=dev)
        self.want = oracle.forward(cfg, w, frames, off, ids, L0=L0, compose=compose)["logits"]

    def run(self, nbytes):
        logits = torch.full((self.R, self.cfg.C), float("nan"), device="cuda")
        status = torch.zeros(1, dtype=torch.int32, device="cuda")
        rc = binding.poly_forward(self.model, self.frames, self.off, self.ids, self.R, torch.empty_like(logits), self.ws[:nbytes], out_logits=logits,
                                  dev_status=status, check=False)
        torch.cuda.synchronize()
        return rc, logits.cpu().numpy(), int(status.item())

    def least(self):
        """The smallest workspace that is taken (sizes are multiples of 256 bytes)."""
        lo, hi = 0, self.ws.numel() // 256
        while hi - lo > 1:
            mid = (lo + hi) // 2
            if mid and self.run(256 * mid)[0] == 0:
                hi = mid
            else:
                lo = mid
        return 256 * hi

    def check(self, nbytes, repeats=1):
        binding.poly_profile_begin(400)
        try:
            rc, got, status = self.run(nbytes)
        finally:
            prof = binding.poly_profile_end()
        assert rc == 0 and status == 0
        assert prof["attention"]["launches"] == self.cfg.L
        assert np.abs(got - self.want).max() < TOL
        for _ in range(repeats):
            assert np.array_equal(got, self.run(nbytes)[1])
        return {n: prof[n]["launches"] for n in prof}


@pytest.mark.parametrize("compose", ["branch", "sum"])
@pytest.mark.parametrize("targets,L0,r", [(15, 0, 4), (3, 1, 8), (12, 0, 16), (5, 2, 4), (10, 2, 20)])
def test_all_target_sets(targets, L0, r, compose):
    case = synth.make_small_case(40 + targets, dtype=synth.DT_BF16, targets=targets, L=3, F=5, r=r, max_set=3, n_adapters=4, hw=48, patch=8)
    call = Call(*case, L0, compose)
    call.check(call.least())


@pytest.mark.parametrize("D,heads,Dm,hw,r,targets,L0", [
    (64, 1, 128, 48, 4, 3, 0),      # one 64-column tile, T = 37: a single ragged row tile
    (64, 1, 192, 64, 16, 1, 1),     # T = 65: a full tile and a one-row tile; adapters on qkv only; fan-out at layer 1
    (128, 2, 256, 64, 12, 3, 0),    # rank 12: the second half of the expand operand is partly empty
    (192, 3, 768, 40, 8, 3, 2),     # DeiT-tiny widths, T = 26, fan-out at layer 2
    (192, 3, 320, 72, 16, 2, 0),    # adapters on proj only, Dm = 5 chunks, T = 82
    (128, 2, 384, 64, 8, 3, 0),     # Dm = 6 chunks: the last feed-forward item and the second qkv item share a stage of the weight ring
])
def test_row_kernel_widths(D, heads, Dm, hw, r, targets, L0):
    case = synth.make_small_case(60 + D + r, dtype=synth.DT_BF16, targets=targets, L=4, F=4, r=r, max_set=3, n_adapters=5, D=D, heads=heads,
                                 Dm=Dm, hw=hw, patch=8)
    call = Call(*case, L0)
    # patch embedding, the first qkv (and the one where frames fan out), one row kernel per layer.  Repeated: a stage of the weight ring that
    # is refilled one step early shows up as run-to-run differences long before it shows up as a wrong answer
    assert call.check(call.least(), repeats=8)["gemm"] == 1 + 1 + (1 if L0 else 0) + 4


@pytest.mark.parametrize("targets,r,L0", [(3, 8, 2), (1, 16, 0)])
def test_summed_terms_of_a_narrow_model(targets, r, L0):
    case = synth.make_small_case(452 + r, dtype=synth.DT_BF16, targets=targets, L=4, F=6, r=r, max_set=3, n_adapters=5, D=192, heads=3, Dm=768,
                                 hw=72, patch=8)
    call = Call(*case, L0, "sum")
    call.check(call.least())


def _many(n, per, n_adapters, seed):
    rng = np.random.default_rng(seed)
    return synth.sets_to_csr([sorted(rng.choice(n_adapters, size=per, replace=False)) for _ in range(n)])


@pytest.mark.parametrize("F", [5, 60])           # the second: 120 blocks of three tiles, more than run as tasks
@pytest.mark.parametrize("L0", [0, 2])
def test_rank_outside_the_row_kernel_runs_the_feed_forward_kernel(F, L0):
    cfg, w, frames, _, _ = synth.make_small_case(140, dtype=synth.DT_BF16, targets=3, L=3, F=F, r=20, max_set=3, n_adapters=4, D=192, heads=3,
                                                 Dm=768, hw=72, patch=8)                       # T = 82: a full and a ragged tile
    call = Call(cfg, w, frames, *_many(F, 2, 4, 1), L0)
    n = call.check(call.ws.numel() if F == 60 and L0 == 0 else call.least())
    if L0 == 0:
        assert n["gemm"] == 1 + 3 * 3 and n["layernorm"] == 3                                  # qkv, proj, feed-forward with its LayerNorm


@pytest.mark.parametrize("compose", ["branch", "sum"])
@pytest.mark.parametrize("targets,r,D,heads,Dm", [
    (12, 16, 192, 3, 768),                       # adapters on fc1 and fc2: the fc1 linear with its GELU in the row-tile kernel
    (15, 4, 128, 2, 384),
    (15, 20, 192, 3, 640),                       # a rank that no row kernel takes: the GEMM path
    (3, 8, 192, 3, 768),                         # summed: the GEMM path
])
def test_more_blocks_than_run_as_tasks(targets, r, D, heads, Dm, compose):
    F, per = (90, 2) if compose == "branch" else (170, 2)
    cfg, w, frames, _, _ = synth.make_small_case(500 + targets + r, dtype=synth.DT_BF16, targets=targets, L=2, F=F, r=r, max_set=2, n_adapters=5,
                                                 D=D, heads=heads, Dm=Dm, hw=48, patch=8)      # T = 37: 360 and 340 tiles
    call = Call(cfg, w, frames, *_many(F, per, 5, 2), 0, compose)
    call.check(call.ws.numel())


@pytest.mark.parametrize("F,compose", [(8, "branch"), (8, "sum"), (48, "branch"), (48, "sum")])
def test_paper_preset(F, compose):
    """Query + value adapters (rank 32 on the fused qkv linear) on the last two layers."""
    cfg, w, frames, off, ids = synth.make_paper_preset(F=F)
    call = Call(cfg, w, frames, off, ids, cfg.L0, compose)
    call.check(call.least() if F == 8 else call.ws.numel())
