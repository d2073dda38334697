"""Many rows of a model 192 wide: tiles of 128 and 256 rows in registers (rowreg.hip) where they, their waves and the blocks in them end."""
import numpy as np
import pytest
import torch

import oracle
from paper_2507_14959_amd import binding, synth

pytestmark = pytest.mark.gpu

UNIQUE = 12                      # different frames; the call repeats them, a row depends on its frame and adapter only
BOUND = 6e-3                     # as for the tiles of 64 rows (test_row_layer.py); 1.0e-3 to 2.5e-3 here


def _case(F, hw, patch, Dm, r, targets, per_frame, L=3, seed=0):
    cfg, w, frames, _, _ = synth.make_small_case(900 + Dm + hw + r + seed, dtype=synth.DT_BF16, targets=targets, L=L, F=UNIQUE, r=r, n_adapters=5, D=192, heads=3,
                                                 Dm=Dm, hw=hw, patch=patch)
    rng = np.random.default_rng(Dm + r)
    sets = [sorted(rng.choice(5, size=1 + f % per_frame, replace=False)) for f in range(UNIQUE)]
    which = np.arange(F) % UNIQUE
    off, ids = synth.sets_to_csr([sets[f] for f in which])
    rows = np.concatenate([[sum(map(len, sets[:f])) + i for i in range(len(sets[f]))] for f in which]).astype(int)
    return cfg, w, frames, sets, frames[which], off, ids, rows


def _want(cfg, w, frames, sets, rows, L0):
    off, ids = synth.sets_to_csr(sets)
    return oracle.forward(cfg, w, frames, off, ids, L0=L0)["logits"][rows]


CASES = [
    (460, 48, 8, 768, 8, 3, 1, 0),        # 37 tokens, 128-row tiles, 28 rows in the last wave
    (300, 48, 8, 128, 16, 3, 2, 0),       # the count only on the device; the shortest hidden width
    (460, 48, 8, 192, 16, 1, 1, 60),      # room for more blocks than there are; adapters on qkv only
    (520, 48, 8, 320, 8, 2, 1, 0),        # on proj only
    (900, 48, 8, 256, 8, 3, 1, 0),        # 256-row tiles, 20 rows in the last of them: waves without any
    (700, 40, 8, 192, 16, 3, 1, 0),       # 26 tokens: by itself a block shorter than a wave's rows keeps the tiles of 64 rows where adapters differ
    (100, 112, 8, 768, 16, 3, 2, 0),      # 197 tokens
]


@pytest.mark.parametrize("F,hw,patch,Dm,r,targets,per_frame,spare", CASES)
@pytest.mark.parametrize("L0", [0, 1, 3])
def test_against_the_oracle(F, hw, patch, Dm, r, targets, per_frame, spare, L0):
    cfg, w, frames, sets, many, off, ids, rows = _case(F, hw, patch, Dm, r, targets, per_frame)
    model = binding.DeviceModel(cfg, w, L0=L0)
    binding.poly_profile_begin(400)
    try:
        got = binding.run_forward(model, many, off, ids, R_cap=len(ids) + spare)
    finally:
        prof = binding.poly_profile_end()
    assert prof["attention"]["launches"] == 3 and prof["layernorm"]["launches"] == 0       # layer by layer, everything between two attentions in a launch
    logits = got["logits"][:len(ids)]
    again = binding.run_forward(model, many, off, ids, R_cap=len(ids) + spare)["logits"][:len(ids)]
    assert got["status"] == 0 and np.array_equal(logits, again)
    assert np.abs(logits - _want(cfg, w, frames, sets, rows, L0)).max() < BOUND
    first = np.unique(rows, return_index=True)[1]
    assert np.array_equal(logits, logits[first[rows]])     # wherever in a tile a block lies


# More than 65 536 rows: 256 tiles of 256 and, in a launch of their own, the rest on tiles of 128.  Frames of 37 tokens, those of them that have an adapter
BOTH = [(1772, 1772), (1900, 1900), (2655, 2655), (1900, 1772), (1900, 1600)]       # 28 rows past, tiles past, 99 rows short of a round and a half; the last pairs not there, all of the rest


@pytest.mark.parametrize("F,n", BOTH)
@pytest.mark.parametrize("L0", [0, 1, 3])
def test_full_rounds_and_the_rows_past_them(F, n, L0):
    cfg, w, frames, sets, many, off, ids, rows = _case(F, 48, 8, 128, 8, 3, 1)
    off, room = np.minimum(off, n), np.concatenate([ids[:n], np.zeros(F - n, dtype=ids.dtype)])
    got = binding.run_forward(binding.DeviceModel(cfg, w, L0=L0), many, off, room, R_cap=F)
    assert got["status"] == 0 and np.isnan(got["logits"][n:]).all()
    logits = got["logits"][:n]
    assert np.abs(logits - _want(cfg, w, frames, sets, rows, L0)[:n]).max() < BOUND
    first = np.unique(rows, return_index=True)[1]
    assert np.array_equal(logits, logits[first[rows[:n]]])


ROOM = [
    (120, 400, 0),       # at one adapter a frame tiles of 64 rows are faster
    (250, 300, 0),
    (460, 1000, 4),      # .. waves of 32
]


@pytest.mark.parametrize("F,spare,taken", ROOM)
def test_much_room_takes_the_kernels_of_few_adapters(F, spare, taken):
    """Room for several blocks a frame and one on every frame: the kernels, and so the bits, of a call without room."""
    cfg, w, frames, sets, many, off, ids, rows = _case(F, 48, 8, 192, 8, 3, 1)
    model = binding.DeviceModel(cfg, w, L0=0)
    tight, roomy = (binding.run_forward(model, many, off, ids, R_cap=len(ids) + n)["logits"][:len(ids)] for n in (0, spare))
    assert np.array_equal(tight, roomy)
    assert np.abs(roomy - _want(cfg, w, frames, sets, rows, 0)).max() < BOUND


def test_summed_shared_layers():
    """Terms summed on a frame's block from layer 2 on: up to there its rows run here, and leave in the order that the GEMM path reads."""
    cfg, w, frames, sets, many, off, ids, rows = _case(480, 48, 8, 256, 8, 3, 2)
    got = binding.run_forward(binding.DeviceModel(cfg, w, L0=2, compose="sum"), many, off, ids)
    o, i = synth.sets_to_csr(sets)
    assert got["status"] == 0
    assert np.abs(got["logits"] - oracle.forward(cfg, w, frames, o, i, L0=2, compose="sum")["logits"][rows]).max() < BOUND


LOOP = (460, 48, 8, 256, 8, 3)   # frames, their size, patch, hidden width, rank, row-blocks a frame that there is room for


@pytest.mark.parametrize("compose,targets,L0,room", [
    ("sum", 0, 1, 3),        # no linear adapted: the row kernels go on past the selection, which reads the rows before they do
    ("sum", 0, 2, 3),
    ("sum", 3, 2, 0),        # no room for a row-block: base scores only
    ("sum", 3, 1, 3),
    ("branch", 3, 1, 3),
    ("branch", 1, 2, 3),
    ("branch", 3, 3, 3),     # no adapted layer
])
def test_the_lagged_loop(compose, targets, L0, room):
    dev = "cuda"
    F, hw, patch, Dm, r, _ = LOOP
    cfg, w, _, _, many, _, _, _ = _case(F, hw, patch, Dm, r, targets, 1)
    K = cfg.n_adapters * cfg.C
    member = synth.make_group_membership(cfg.n_adapters, cfg.C)
    cap, theta = room * F, 0.5 if room else 2.0            # (without room no label may be on)
    bw, bb = synth.make_base_head(cfg, K, 17, bias_mean=-3.5)
    model = binding.DeviceModel(cfg, w, L0=L0, compose=compose)
    head = binding.DeviceStream(model, bw, bb, member, theta=theta)
    off, ids, cnt, status = (torch.zeros(n, dtype=torch.int32, device=dev) for n in (F + 1, max(cap, 1), 2, 1))
    scores, logits = (torch.zeros(max(cap, 1), cfg.C, device=dev) for _ in range(2))
    base = torch.zeros(F, K, device=dev)
    ws = torch.empty(binding.poly_stream_step_workspace_bytes(model, F, cap, K), dtype=torch.uint8, device=dev)
    binding.poly_stream_step(model, head, model.frames_to_device(many), cap, off, ids, cnt, scores, ws, out_base_scores=base, out_logits=logits, dev_status=status)
    off, ids, base, logits = (t.cpu().numpy() for t in (off, ids, base, logits))
    want = oracle.base_head(cfg, w, many[:UNIQUE], bw, bb, L0)
    assert int(status.item()) == 0 and np.abs(base - want[np.arange(F) % UNIQUE]).max() < 2e-2          # (test_gpu_stream.py's bound of a score)
    assert np.array_equal(head.carry.cpu().numpy(), base[-1])
    set_off, set_ids, _ = oracle.select(np.concatenate([np.zeros((1, K), np.float32), base[:-1]]), member, theta=theta)
    assert np.array_equal(off, set_off) and np.array_equal(ids[:off[-1]], set_ids) and (off[-1] > 0) == (cap > 0)
    a, b = UNIQUE, 2 * UNIQUE                              # (the first frame has no labels yet)
    got = logits[off[a]:off[b]]
    o, i = off[a:b + 1] - off[a], ids[off[a]:off[b]]
    if cap:
        assert np.abs(got - oracle.forward(cfg, w, many[a:b], o, i, L0=L0, compose=compose)["logits"]).max() < BOUND


def test_an_adapter_stays_with_its_blocks():
    """Two blocks in a wave's rows: infinities of one block's adapter do not reach the other's rows."""
    cfg, w, frames, sets, many, off, ids, rows = _case(460, 48, 8, 192, 8, 3, 1)
    clean = binding.run_forward(binding.DeviceModel(cfg, w, L0=0), many, off, ids)["logits"]
    bad = dict(w, B_qkv=np.array(w["B_qkv"]), A_proj=np.array(w["A_proj"]))
    bad["B_qkv"][:, 3] = np.inf
    bad["A_proj"][:, 3] = -np.inf
    got = binding.run_forward(binding.DeviceModel(cfg, bad, L0=0), many, off, ids)["logits"]
    other = np.asarray(ids) != 3
    assert 0 < other.sum() < len(ids)
    assert np.array_equal(got[other], clean[other]) and not np.isfinite(got[~other]).any()
