"""Runs of layers on tiles of 64 or 32 rows that stay on their CUs: edges of tiles and key tiles, ranks and targets, several rounds, launches that share the layers, stalls."""
from dataclasses import replace

import numpy as np
import pytest
import torch

import oracle
from paper_2507_14959_amd import binding, synth

pytestmark = pytest.mark.gpu

TOL = 8e-3          # bf16 activations between the steps; test_gpu_flow_sizes.py holds the same layers as tasks to it


def _case(T, F, Dm, r, targets, L, per_frame, seed):
    """T - 1 patches of 8 in a row, F frames of which 8 differ, up to per_frame adapters on a frame."""
    cfg, _, _, _, _ = synth.make_small_case(seed, dtype=synth.DT_BF16, targets=targets, L=L, F=1, r=r, n_adapters=5, D=192, heads=3, Dm=Dm, hw=16, patch=8)
    cfg = replace(cfg, H=8, W=8 * (T - 1))
    rng = np.random.default_rng(seed)
    w, eight = synth.make_weights(cfg, rng), synth.make_frames(cfg, 8, rng)
    sets = [np.sort(rng.choice(5, size=1 + f % per_frame, replace=False)) for f in range(8)]
    pick = np.arange(F) % 8
    return cfg, w, eight, sets, eight[pick], *synth.sets_to_csr([sets[p] for p in pick])


def _compare(cfg, eight, sets, got, w, L0, off):
    off8, ids8 = synth.sets_to_csr(sets)
    want = oracle.forward(cfg, w, eight, off8, ids8, L0=L0)["logits"]
    rows = np.concatenate([np.arange(off8[f % 8], off8[f % 8 + 1]) for f in range(len(off) - 1)])
    err = np.abs(got - want[rows]).max()
    print(f"logits max-abs error {err:.2e} of up to {np.abs(want).max():.2f}")
    assert err < TOL


# rows of a tile in the adapted layers, T, frames, hidden width, rank, targets (1 qkv, 2 proj), layers, first adapted layer, adapters a frame up to, spare room
CASES = [
    (32, 17, 100, 128, 8, 3, 4, 0, 1, 0),       # a tile a block, the second half of the keys empty, one chunk of hidden columns
    (32, 33, 40, 192, 4, 1, 5, 1, 2, 0),        # half a chunk; a row in the second tile, which is the second half of the keys; qkv alone
    (32, 64, 50, 768, 12, 2, 4, 0, 1, 0),       # whole tiles; proj alone
    (32, 65, 30, 256, 16, 3, 4, 2, 2, 25),      # two key tiles of four with a row in the second half; room for more than there is
    (32, 97, 33, 320, 8, 3, 4, 4, 1, 0),        # no adapted layer; three chunks, the last half a one
    (32, 128, 20, 384, 8, 3, 4, 0, 1, 0),
    (32, 129, 24, 192, 16, 3, 4, 0, 2, 10),     # five key tiles of seven
    (32, 224, 10, 192, 4, 3, 4, 2, 1, 0),       # the most tokens
    (32, 70, 140, 128, 8, 3, 4, 0, 1, 0),       # 420 tiles, three a block: two rounds of 80 blocks
    (64, 64, 140, 128, 8, 3, 4, 0, 1, 0),       # a whole tile a block
    (64, 65, 90, 256, 16, 3, 4, 2, 2, 0),       # one row in a block's second tile
    (64, 97, 70, 320, 8, 3, 4, 0, 1, 10),
    (64, 170, 44, 128, 8, 3, 4, 1, 1, 0),       # three tiles, six key tiles
    (64, 193, 38, 768, 8, 3, 4, 0, 1, 6),       # one row in the fourth tile
    (64, 197, 75, 192, 8, 3, 4, 0, 1, 0),       # 300 tiles: a second round
    (64, 224, 40, 192, 4, 1, 4, 2, 1, 0),
    (64, 197, 64, 128, 8, 3, 4, 2, 3, 100),     # a bound of four a frame, more than 512 tiles of what is usual
    (32, 20, 520, 128, 8, 3, 4, 0, 1, 0),       # three rounds of blocks too short for rowreg.hip
]


@pytest.mark.parametrize("rows,T,F,Dm,r,targets,L,L0,per_frame,spare", CASES)
def test_against_the_oracle(rows, T, F, Dm, r, targets, L, L0, per_frame, spare):
    cfg, w, eight, sets, frames, off, ids = _case(T, F, Dm, r, targets, L, per_frame, 2000 + T + rows)
    model = binding.DeviceModel(cfg, w, L0=L0)
    binding.poly_profile_begin(400)
    try:
        got = binding.run_forward(model, frames, off, ids, R_cap=int(off[-1]) + spare)
    finally:
        prof = binding.poly_profile_end()
    assert prof["attention"]["launches"] == 0
    again = binding.run_forward(model, frames, off, ids, R_cap=int(off[-1]) + spare)
    n = int(off[-1])
    assert got["status"] == 0 and np.array_equal(got["logits"][:n], again["logits"][:n])
    assert np.isnan(got["logits"][n:]).all()
    _compare(cfg, eight, sets, got["logits"][:n], w, L0, off)
    _same_wherever_a_frame_sits(got["logits"], off)


def _run_of_tiles(model, frames, off, ids, **kw):
    """run_forward, where all layers run as launches of many and one of them is too large for the small tasks."""
    binding.poly_profile_begin(400)
    try:
        got = binding.run_forward(model, frames, off, ids, **kw)
    finally:
        prof = binding.poly_profile_end()
    assert prof["attention"]["launches"] == 0 and (len(off) - 1) * ((model.cfg.T + 31) // 32) > 44     # (FLOW_FEW)
    return got


def _same_wherever_a_frame_sits(logits, off):
    for f in range(8, len(off) - 1):
        assert np.array_equal(logits[off[f]:off[f + 1]], logits[off[f % 8]:off[f % 8 + 1]])


def _forward(model, frames, off, ids, ws, room):
    dev = "cuda"
    out = torch.full((room, model.cfg.C), float("nan"), device=dev)
    status = torch.full((1,), 99, dtype=torch.int32, device=dev)
    binding.poly_profile_begin(400)
    try:
        rc = binding.poly_forward(model, model.frames_to_device(frames), torch.from_numpy(off).to(dev, torch.int32), torch.from_numpy(ids).to(dev, torch.int32),
                                  room, torch.zeros_like(out), ws, out_logits=out, dev_status=status, check=False)
    finally:
        prof = binding.poly_profile_end()
    return rc, out.cpu().numpy(), int(status.item()), prof


# several: the smaller workspaces take another number of launches (with room for as many blocks again as there are)
@pytest.mark.parametrize("T,F,room,L0,several", [(50, 60, 120, 0, True), (50, 60, 60, 0, False), (113, 40, 100, 4, False), (197, 20, 40, 0, False)])
def test_the_launches_share_the_layers_without_changing_a_bit(T, F, room, L0, several):
    cfg, w, eight, sets, frames, off, ids = _case(T, F, 128, 8, 3, 12, 1, 3000 + T)
    model = binding.DeviceModel(cfg, w, L0=L0)
    full = torch.empty(binding.poly_forward_workspace_bytes(model, F, room), dtype=torch.uint8, device="cuda")
    first, launches = None, set()
    for part in range(24, 8, -1):
        ws = full[:full.numel() * part // 24 // 256 * 256]
        ws.fill_(0xff)
        rc, got, status, prof = _forward(model, frames, off, ids, ws, room)
        if rc == binding.POLY_ECAP:
            break
        assert rc == 0 and status == 0
        if prof["attention"]["launches"] == 0:
            first = got if first is None else first
            assert np.array_equal(got, first, equal_nan=True)
            launches.add(prof["gemm"]["launches"])
        else:
            assert np.nanmax(np.abs(got - first)) < TOL
    print(f"launches of the product stage {sorted(launches)}")
    assert first is not None and (len(launches) > 1 or not several)
    _compare(cfg, eight, sets, first[:F], w, L0, off)


@pytest.mark.parametrize("L0", [0, 2, 5])
def test_a_stall_is_reported_and_nothing_published(L0):
    cfg, w, eight, sets, frames, off, ids = _case(197, 12, 128, 8, 3, 5, 1, 4000)
    model = binding.DeviceModel(cfg, w, L0=L0)
    want = _run_of_tiles(model, frames, off, ids)
    binding.lib().poly_wait_limit(0)
    try:
        got = binding.run_forward(model, frames, off, ids)
    finally:
        binding.lib().poly_wait_limit(-1)
    assert got["status"] == binding.POLY_ESTALL and np.isnan(got["logits"]).all()
    got = binding.run_forward(model, frames, off, ids)
    assert got["status"] == 0 and np.array_equal(got["logits"], want["logits"])
    _compare(cfg, eight, sets, got["logits"], w, L0, off)


# as many workgroups as a block has tiles; one fewer than may start at eight queues, as many
@pytest.mark.parametrize("T,F,L0,compose,tiles", [(197, 40, 2, "branch", 4), (197, 12, 0, "branch", 7), (113, 24, 0, "sum", 4), (65, 26, 0, "branch", 3), (193, 7, 4, "branch", 7)])
def test_few_workgroups_come_to_the_end(T, F, L0, compose, tiles):
    """Where few CUs are free: no more blocks are begun than the workgroups that are there can finish."""
    cfg, w, eight, sets, frames, off, ids = _case(T, F, 128, 8, 3, 4, 1, 4200 + T)
    model = binding.DeviceModel(cfg, w, L0=L0, compose=compose)
    want = _run_of_tiles(model, frames, off, ids)
    enough = min(F, 8) * (tiles - 1) + 1
    for workgroups in (tiles, enough - 1, enough):
        binding.lib().poly_wait_workgroups(workgroups)
        try:
            got = binding.run_forward(model, frames, off, ids)
        finally:
            binding.lib().poly_wait_workgroups(0)
        assert got["status"] == 0 and np.array_equal(got["logits"], want["logits"]), workgroups
    binding.lib().poly_wait_workgroups(tiles - 1)
    binding.lib().poly_wait_limit(2000)
    try:
        got = binding.run_forward(model, frames, off, ids)
    finally:
        binding.lib().poly_wait_workgroups(0)
        binding.lib().poly_wait_limit(-1)
    assert got["status"] == binding.POLY_ESTALL and np.isnan(got["logits"]).all()


def test_a_bad_adapter_id_computes_nothing():
    cfg, w, eight, sets, frames, off, ids = _case(113, 40, 128, 8, 3, 4, 1, 4100)
    model = binding.DeviceModel(cfg, w, L0=0)
    _run_of_tiles(model, frames, off, ids)
    ids = ids.copy()
    ids[7] = 5
    got = binding.run_forward(model, frames, off, ids)
    assert got["status"] == binding.POLY_ERANGE and np.isnan(got["logits"]).all()


# The sum of a block's terms: none, one, up to four in LDS (two of rank 16, three of 12), more than have a place there; a second round
@pytest.mark.parametrize("T,F,Dm,r,targets,L,L0,most", [(17, 100, 128, 8, 3, 4, 0, 2), (50, 40, 192, 4, 1, 4, 1, 4), (113, 24, 256, 16, 3, 4, 0, 4), (197, 12, 128, 12, 2, 4, 2, 5),
                                                        (97, 30, 768, 8, 3, 4, 0, 8), (224, 40, 128, 8, 3, 4, 0, 3)])
def test_summed_terms(T, F, Dm, r, targets, L, L0, most):
    cfg, w, eight, _, frames, _, _ = _case(T, F, Dm, r, targets, L, 1, 5000 + T)
    cfg = replace(cfg, n_adapters=9)
    rng = np.random.default_rng(T)
    w = synth.make_weights(cfg, rng)
    sets = [np.sort(rng.choice(9, size=f % (most + 1), replace=False)) for f in range(8)]
    off, ids = synth.sets_to_csr([sets[f % 8] for f in range(F)])
    model = binding.DeviceModel(cfg, w, L0=L0, compose="sum")
    binding.poly_profile_begin(400)
    try:
        got = binding.run_forward(model, frames, off, ids)
    finally:
        prof = binding.poly_profile_end()
    assert got["status"] == 0 and prof["attention"]["launches"] == 0
    off8, ids8 = synth.sets_to_csr(sets)
    want = oracle.forward(cfg, w, eight, off8, ids8, L0=L0, compose="sum")["logits"]
    rows = np.concatenate([np.arange(off8[f % 8], off8[f % 8 + 1]) for f in range(F)])
    assert np.abs(got["logits"] - want[rows]).max() < TOL
    _same_wherever_a_frame_sits(got["logits"], off)


def test_two_calls_at_a_time_on_two_streams():
    """Workgroups of two launches share the CUs, so that a block's may have to wait for the other call's to end: the same bits as one after the other."""
    calls = []
    for T, F in ((197, 30), (197, 64)):
        cfg, w, eight, sets, frames, off, ids = _case(T, F, 768, 8, 3, 6, 1, 8000 + F)
        model = binding.DeviceModel(cfg, w, L0=2)
        _run_of_tiles(model, frames, off, ids)
        up = lambda a: torch.from_numpy(a).to("cuda", torch.int32)  # noqa: E731
        ws = torch.empty(binding.poly_forward_workspace_bytes(model, F, F), dtype=torch.uint8, device="cuda")
        calls.append((model, model.frames_to_device(frames), up(off), up(ids), F, ws, torch.cuda.Stream()))

    def run(call, outs, status):
        model, frames, off, ids, F, ws, _ = call
        binding.poly_forward(model, frames, off, ids, F, torch.empty_like(outs), ws, out_logits=outs, dev_status=status)

    fresh = lambda c: (torch.full((c[4], c[0].cfg.C), float("nan"), device="cuda"), torch.full((1,), 99, dtype=torch.int32, device="cuda"))  # noqa: E731
    alone = [fresh(c) for c in calls]
    for c, (o, s) in zip(calls, alone):
        run(c, o, s)
    torch.cuda.synchronize()
    got = [[fresh(c) for _ in range(8)] for c in calls]
    torch.cuda.synchronize()
    for i in range(8):
        for c, outs in zip(calls, got):
            with torch.cuda.stream(c[6]):
                run(c, *outs[i])
    torch.cuda.synchronize()
    for (want, st), outs in zip(alone, got):
        assert int(st.item()) == 0
        for o, s in outs:
            assert int(s.item()) == 0 and torch.equal(o, want)


def test_a_captured_call_replays():
    """The counters are cleared by the call's first kernel, so every replay starts from nothing; other frames in the same buffer in between."""
    cfg, w, eight, sets, frames, off, ids = _case(113, 40, 768, 8, 3, 6, 1, 8200)
    model = binding.DeviceModel(cfg, w, L0=2)
    _run_of_tiles(model, frames, off, ids)
    F = len(frames)
    up = lambda a: torch.from_numpy(a).to("cuda", torch.int32)  # noqa: E731
    src = [model.frames_to_device(f) for f in (frames, np.ascontiguousarray(frames[::-1]))]
    buf, off_d, ids_d = src[0].clone(), up(off), up(ids)
    ws = torch.empty(binding.poly_forward_workspace_bytes(model, F, F), dtype=torch.uint8, device="cuda")
    scores, logits = (torch.zeros(F, cfg.C, device="cuda") for _ in range(2))
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    call = lambda: binding.poly_forward(model, buf, off_d, ids_d, F, scores, ws, out_logits=logits, dev_status=status)  # noqa: E731
    want = []
    for f in src:
        buf.copy_(f)
        call()
        torch.cuda.synchronize()
        want.append(logits.clone())
    assert not torch.equal(*want)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call()
    for i in (0, 1, 1, 0, 1):
        buf.copy_(src[i])
        logits.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert int(status.item()) == 0 and torch.equal(logits, want[i])


def test_a_launch_without_layers_reports_nothing():
    """Room for twice the blocks there are: the host counts two launches by it, the first does all layers.  The second must not read what other workgroups left
    in LDS: those of calls without patience, on another stream meanwhile, leave a count of looks that means a stall."""
    cfg, w, eight, sets, frames, off, ids = _case(50, 60, 128, 8, 3, 12, 1, 8400)
    model = binding.DeviceModel(cfg, w, L0=0)
    F, room = 60, 120
    full = torch.empty(binding.poly_forward_workspace_bytes(model, F, room), dtype=torch.uint8, device="cuda")
    _, want, status, prof = _forward(model, frames, off, ids, full, room)
    assert status == 0 and prof["attention"]["launches"] == 0
    one, ws = prof["gemm"]["launches"], None
    for part in range(24, 8, -1):
        ws = full[:full.numel() * part // 24 // 256 * 256]
        _, got, status, prof = _forward(model, frames, off, ids, ws, room)
        assert status == 0 and prof["attention"]["launches"] == 0
        if prof["gemm"]["launches"] > one:
            break
    assert prof["gemm"]["launches"] > one and np.array_equal(got, want, equal_nan=True)

    up = lambda a: torch.from_numpy(a).to("cuda", torch.int32)  # noqa: E731
    src, off_d, ids_d, other = model.frames_to_device(frames), up(off), up(ids), torch.empty_like(full)
    calls = [(torch.full((room, cfg.C), float("nan"), device="cuda"), torch.full((1,), 99, dtype=torch.int32, device="cuda")) for _ in range(24)]
    lost, stalled = torch.zeros(room, cfg.C, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
    mine, theirs = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    for logits, st in calls:
        try:
            binding.lib().poly_wait_limit(0)
            with torch.cuda.stream(theirs):
                for _ in range(2):
                    binding.poly_forward(model, src, off_d, ids_d, room, torch.empty_like(lost), other, out_logits=lost, dev_status=stalled)
        finally:
            binding.lib().poly_wait_limit(-1)
        with torch.cuda.stream(mine):
            binding.poly_forward(model, src, off_d, ids_d, room, torch.empty_like(logits), ws, out_logits=logits, dev_status=st)
    torch.cuda.synchronize()
    assert int(stalled.item()) == binding.POLY_ESTALL
    for logits, st in calls:
        assert int(st.item()) == 0 and np.array_equal(logits.cpu().numpy(), want, equal_nan=True)
