"""Attention of long blocks with two query tiles per wave: more (block, head) pairs than CUs."""
import numpy as np
import pytest
import torch

import oracle
import test_gpu_rowrun as run
from paper_2507_14959_amd import binding, synth
from test_gpu_forward import compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,heads,Dm,hw,F,L0", [
    (64, 1, 128, 104, 270, 1),       # 170 tokens: six query tiles on three waves, ten rows in the last
    (128, 2, 128, 112, 135, 1),      # 197 tokens: seven on four, one wave with a single tile
    (256, 4, 256, 112, 65, 1),       # the wide path
    (64, 1, 128, 112, 250, 1),       # frames on one side of the rule, their branches on the other
])
def test_against_the_oracle(D, heads, Dm, hw, F, L0):
    cfg, w, frames, off, ids = synth.make_small_case(7 + D + hw, dtype=synth.DT_BF16, targets=3, L=2, F=F, r=8, max_set=2, n_adapters=5, D=D, heads=heads,
                                                     Dm=Dm, hw=hw, patch=8)
    compare(cfg, w, frames, off, ids, L0, tol=6e-3)          # (0.8e-3 to 2.1e-3; a bias left out of one linear of a layer: 9.5e-3 and more)


@pytest.mark.parametrize("hw,n,adapters,cap", [
    (112, 100, 1, 400),      # 200 pairs of a bound of 800: a tile per wave
    (112, 100, 2, 200),      # 400 pairs: half the waves leave, one of the others has a single tile
    (112, 128, 1, 512),      # 256 pairs, the last count of a tile per wave
    (112, 43, 3, 172),       # 258 pairs
    (104, 100, 2, 300),      # 170 tokens: six tiles
    (104, 90, 1, 360),
])
def test_form_by_the_true_count(hw, n, adapters, cap):
    """Room for more adapters than are in use, and frames on the small side of the rule: which form runs is the device's choice."""
    cfg, w, frames, _, _ = synth.make_small_case(900 + n + hw, dtype=synth.DT_BF16, targets=3, L=2, F=n, r=8, n_adapters=5, D=128, heads=2, Dm=128, hw=hw,
                                                 patch=8)
    rng = np.random.default_rng(n)
    off, ids = synth.sets_to_csr([sorted(rng.choice(5, size=adapters, replace=False)) for _ in range(n)])
    room = np.concatenate([ids, np.zeros(cap - len(ids), dtype=ids.dtype)])
    got = binding.run_forward(binding.DeviceModel(cfg, w, L0=0), frames, off, room, R_cap=cap)
    want = oracle.forward(cfg, w, frames, off, ids, L0=0)["logits"]
    # 1.1e-3 to 1.7e-3 over the cases; a linear's bias left out of one layer moves the logits by 6e-3 and more
    assert got["status"] == 0 and np.abs(got["logits"][:len(ids)] - want).max() < 4e-3


# Keys have a place in LDS 16 at a time, tiles are 32: the second half of the last tile there or not, by one key, in every number of tiles, on two workgroups a head, one and fewer waves
@pytest.mark.parametrize("F", [40, 60, 150])
@pytest.mark.parametrize("T", [2, 16, 17, 32, 33, 48, 49, 64, 80, 81, 112, 113, 144, 145, 176, 177, 192, 193, 208, 209, 224])
def test_the_last_tile_of_keys(T, F):
    cfg, w, eight, sets, frames, off, ids = run._case(T, F, 128, 8, 3, 3, 1, 7000 + T)
    model = binding.DeviceModel(cfg, w, L0=0)
    ws = torch.empty(binding.poly_forward_workspace_bytes(model, F, F), dtype=torch.uint8, device="cuda")
    lo, hi = 0, ws.numel() // 256
    while hi - lo > 1:                                       # the smallest workspace that is taken: layer by layer
        mid = (lo + hi) // 2
        lo, hi = (lo, mid) if run._forward(model, frames, off, ids, ws[:256 * mid], F)[0] == 0 else (mid, hi)
    rc, got, status, prof = run._forward(model, frames, off, ids, ws[:256 * hi], F)
    assert rc == 0 and status == 0 and prof["attention"]["launches"] == 3
    run._compare(cfg, eight, sets, got, w, 0, off)
    run._same_wherever_a_frame_sits(got, off)
