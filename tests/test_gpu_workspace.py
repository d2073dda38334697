"""One workspace for calls of several sizes, and workspaces smaller than the size the library names, on the GPU."""
import numpy as np
import pytest
import torch

import oracle
from paper_2507_14959_amd import binding, synth

pytestmark = pytest.mark.gpu

TOL = 2e-2
MODEL = dict(dtype=synth.DT_BF16, L=12, n_adapters=4, D=64, heads=1, Dm=128, hw=48, patch=8)      # T = 37: two tiles of 32 rows a block


def _forward(model, frames_np, off, ids, ws):
    dev = "cuda"
    R = int(off[-1])
    frames = model.frames_to_device(frames_np)
    o = torch.from_numpy(off).to(dev, torch.int32)
    i = torch.from_numpy(ids).to(dev, torch.int32)
    out = torch.full((max(R, 1), model.cfg.C), float("nan"), device=dev)
    scores = torch.full_like(out, float("nan"))
    status = torch.full((1,), 99, dtype=torch.int32, device=dev)
    binding.poly_profile_begin(400)
    try:
        rc = binding.poly_forward(model, frames, o, i, R, scores, ws, out_logits=out, dev_status=status, check=False)
    finally:
        prof = binding.poly_profile_end()
    return rc, out.cpu().numpy()[:R], int(status.item()), prof


def _sets(n, per, n_adapters, seed):
    rng = np.random.default_rng(seed)
    return synth.sets_to_csr([sorted(rng.choice(n_adapters, size=per, replace=False)) for _ in range(n)])


@pytest.mark.parametrize("compose", ["branch", "sum"])
@pytest.mark.parametrize("L0,targets,r", [(0, 3, 8), (10, 15, 8), (5, 1, 16)])
def test_workspace_of_the_largest_call_serves_the_smaller_ones(L0, targets, r, compose):
    """The largest call has too many blocks for the task queue, the smaller ones have not."""
    cfg, w, frames, _, _ = synth.make_small_case(700 + L0, F=90, targets=targets, r=r, max_set=2, **MODEL)
    model = binding.DeviceModel(cfg, w, L0=L0, compose=compose)
    ws = torch.empty(binding.poly_forward_workspace_bytes(model, 90, 180), dtype=torch.uint8, device="cuda")
    for F, per in ((90, 2), (30, 2), (20, 2), (60, 1), (1, 1), (90, 2)):
        off, ids = _sets(F, per, cfg.n_adapters, F)
        ws.fill_(0xff)                                       # nothing an earlier call left behind may be needed
        rc, got, status, _ = _forward(model, frames[:F], off, ids, ws)
        assert rc == 0 and status == 0
        n = min(F, 12)
        o1, i1 = off[:n + 1], ids[:off[n]]
        want = oracle.forward(cfg, w, frames[:n], o1, i1, L0=L0, compose=compose)
        assert np.abs(got[:off[n]] - want["logits"]).max() < TOL and np.isfinite(got).all()


@pytest.mark.parametrize("L0", [0, 7])
def test_smaller_workspaces_take_fewer_layers_per_launch_then_the_row_kernels(L0):
    cfg, w, frames, _, _ = synth.make_small_case(720 + L0, F=16, targets=3, r=8, max_set=2, **MODEL)
    off, ids = _sets(16, 2, cfg.n_adapters, 3)
    model = binding.DeviceModel(cfg, w, L0=L0)
    want = oracle.forward(cfg, w, frames, off, ids, L0=L0)["logits"]
    full = torch.empty(binding.poly_forward_workspace_bytes(model, 16, 32), dtype=torch.uint8, device="cuda")
    routes, first, refused = set(), None, False
    for part in range(40, 0, -1):
        ws = full[:full.numel() * part // 40]
        ws.fill_(0xff)
        rc, got, status, prof = _forward(model, frames, off, ids, ws)
        if rc == binding.POLY_ECAP:
            refused = True
            assert np.isnan(got).all() and prof["gemm"]["launches"] == 0
            continue
        assert rc == 0 and status == 0 and not refused       # once too small, always too small
        assert np.abs(got - want).max() < TOL
        tasks = prof["attention"]["launches"] == 0           # every layer as tasks, whatever the number of launches: the same bits
        if tasks:
            first = got if first is None else first
            assert np.array_equal(got, first)
        routes.add((prof["gemm"]["launches"], prof["attention"]["launches"]))
    assert refused and first is not None
    assert sum(a == 0 for _, a in routes) >= 2 and any(a == cfg.L for _, a in routes)      # one launch, several, none as tasks


def test_stream_step_workspace_of_the_largest_call():
    n_ad, gsz = 4, 3
    K = n_ad * gsz
    cfg, w, frames, _, _ = synth.make_small_case(740, F=90, targets=3, r=8, max_set=2, **{**MODEL, "n_adapters": n_ad})
    cfg_w = dict(w)
    model = binding.DeviceModel(cfg, cfg_w, L0=10)
    bw, bb = synth.make_base_head(cfg, K, 9)
    dev = "cuda"
    ws = torch.empty(binding.poly_stream_step_workspace_bytes(model, 90, 360, K), dtype=torch.uint8, device=dev)

    def step(F, cap, space):
        s = binding.DeviceStream(model, bw, bb, synth.make_group_membership(n_ad, gsz))
        off = torch.zeros(F + 1, dtype=torch.int32, device=dev)
        ids = torch.zeros(cap, dtype=torch.int32, device=dev)
        cnt = torch.zeros(2, dtype=torch.int32, device=dev)
        st = torch.zeros(1, dtype=torch.int32, device=dev)
        scores = torch.zeros(cap, cfg.C, device=dev)
        base = torch.zeros(F, K, device=dev)
        binding.poly_stream_step(model, s, model.frames_to_device(frames[:F]), cap, off, ids, cnt, scores, space, out_base_scores=base, dev_status=st)
        torch.cuda.synchronize()
        assert int(st.item()) == 0
        return [t.cpu().numpy() for t in (off, ids, cnt, scores, base, s.carry)]

    for F in (90, 3, 17):
        own = torch.empty(binding.poly_stream_step_workspace_bytes(model, F, 4 * F, K), dtype=torch.uint8, device=dev)
        for a, b in zip(step(F, 4 * F, ws), step(F, 4 * F, own)):
            assert np.array_equal(a, b)
