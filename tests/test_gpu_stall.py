"""The task queue's bounded wait: with no patience at all, every kernel still ends, the call reports POLY_ESTALL and publishes nothing."""
import numpy as np
import pytest
import torch

import oracle
from paper_2507_14959_amd import binding, synth

pytestmark = pytest.mark.gpu


@pytest.fixture
def no_patience():
    def set_limit(looks):
        binding.lib().poly_wait_limit(looks)
    yield set_limit
    set_limit(-1)


def _model(seed, L0, compose="branch", **kw):
    cfg, w, frames, off, ids = synth.make_small_case(seed, dtype=synth.DT_BF16, targets=3, L=6, F=6, r=8, max_set=2, n_adapters=4, D=128,
                                                      heads=2, Dm=256, hw=48, patch=8, **kw)
    return cfg, w, frames, off, ids, binding.DeviceModel(cfg, w, L0=L0, compose=compose)


@pytest.mark.parametrize("L0,compose", [(0, "branch"), (3, "branch"), (6, "branch"), (2, "sum")])
def test_forward_reports_a_stall_and_writes_no_row(no_patience, L0, compose):
    cfg, w, frames, off, ids, model = _model(810, L0, compose)
    assert len(ids)
    no_patience(0)
    got = binding.run_forward(model, frames, off, ids, K=cfg.n_adapters * cfg.C)
    assert got["status"] == binding.POLY_ESTALL and "waiting" in binding.status_string(got["status"])
    assert np.isnan(got["logits"]).all() and np.isnan(got["scores"]).all() and not got["merged"].any()
    no_patience(-1)
    got = binding.run_forward(model, frames, off, ids)
    want = oracle.forward(cfg, w, frames, off, ids, L0=L0, compose=compose)
    assert got["status"] == 0 and np.abs(got["logits"] - want["logits"]).max() < 2e-2


@pytest.mark.parametrize("L0", [0, 3, 6])
def test_stream_step_reports_a_stall_and_keeps_what_it_carries(no_patience, L0):
    n_ad, gsz, F, dev = 4, 3, 6, "cuda"
    K = n_ad * gsz
    cfg, w, frames, _, _, model = _model(820, L0, C=gsz)
    bw, bb = synth.make_base_head(cfg, K, 9)
    s = binding.DeviceStream(model, bw, bb + 6.0, synth.make_group_membership(n_ad, gsz))     # every label on from the second frame on
    fr = model.frames_to_device(frames)
    off = torch.zeros(F + 1, dtype=torch.int32, device=dev)
    ids = torch.zeros(4 * F, dtype=torch.int32, device=dev)
    cnt = torch.zeros(2, dtype=torch.int32, device=dev)
    st = torch.zeros(1, dtype=torch.int32, device=dev)
    scores = torch.full((4 * F, cfg.C), float("nan"), device=dev)
    ws = torch.empty(binding.poly_stream_step_workspace_bytes(model, F, 4 * F, K), dtype=torch.uint8, device=dev)

    def step():
        binding.poly_stream_step(model, s, fr, 4 * F, off, ids, cnt, scores, ws, dev_status=st)
        torch.cuda.synchronize()
        return int(st.item())

    no_patience(0)
    assert step() == binding.POLY_ESTALL and torch.isnan(scores).all()
    # where the shared layers already run as tasks nothing that the next call starts from may come from them
    if L0 > 0:
        assert not s.state.any() and not s.carry.any()
    no_patience(-1)
    s.state.zero_(), s.carry.zero_()
    assert step() == 0 and int(cnt[0]) == n_ad * (F - 1) and torch.isfinite(scores[:int(cnt[0])]).all() and s.carry.any()
