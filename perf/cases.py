"""Workloads whose speed is tracked: what a program that uses this library has it do, through its public entry points.

Four kinds of call:

  select   poly_select: label scores of consecutive frames -> adapter set of every frame
  stream   poly_stream_step: the lagged loop on live frames (shared layers, base head, selection, adapted layers, heads, merge)
  forward  poly_select + poly_forward + merge on a batch whose label scores are already known
  linear   poly_lora_linear: one multi-adapter linear on its own

Models are the ones of paper_2507_14959_amd.synth: "fp32" (config 1: two layers in single precision), "tiny" (config 2), "preset"
(the paper's trained setting on the same backbone: query + value adapters of rank 16, adapted layers at the end) and "base"
(config 3).  A model's weights are drawn once per process, as a program loads its checkpoint once; frames, label scores, adapter
sets, linear operands and base heads come from the seed.
"""
from __future__ import annotations

import functools
import math
from dataclasses import replace

import numpy as np
import torch

from paper_2507_14959_amd import binding, synth

DEV = "cuda"
GROUP = 5                      # labels per context of the label streams
CONTEXTS = 16


def listed():
    return [
        # one camera batch of the label stream: the smallest call there is, launch and latency only
        dict(name="select_64", kind="select", frames=64, overlap=False, copy=False),
        # a recorded clip in one call: overlapping contexts, accuracy table and context copy, where frames depend on each other
        dict(name="select_1024_overlap", kind="select", frames=1024, overlap=True, copy=True),
        # live video, one frame at a time: the latency a camera sees, in the paper's setting
        dict(name="stream_preset_1", kind="stream", model="preset", height=224, width=224, frames=1, active=2),
        # the same loop on a batch of frames, adapters on the last fifth of the layers
        dict(name="stream_tiny_64", kind="stream", model="tiny", height=224, width=224, frames=64, active=2),
        # single precision (config 1): parity and debugging runs
        dict(name="forward_fp32_4", kind="forward", model="fp32", height=64, width=64, frames=4, adapters=2, first=0, sum=False),
        # config 2, the default workload of bench.py: every layer adapted
        dict(name="forward_tiny_32", kind="forward", model="tiny", height=224, width=224, frames=32, adapters=3, first=0, sum=False),
        # many cameras at once, the paper's placement; an odd number of frames
        dict(name="forward_tiny_333", kind="forward", model="tiny", height=224, width=224, frames=333, adapters=3, first=10, sum=False),
        # several adapters summed on one hidden state, wide frames (8 x 14 patches: 113 tokens, no multiple of any tile)
        dict(name="forward_tiny_sum_24", kind="forward", model="tiny", height=128, width=224, frames=24, adapters=3, first=0, sum=True),
        # a few frames through the large backbone
        dict(name="forward_base_3", kind="forward", model="base", height=224, width=224, frames=3, adapters=3, first=10, sum=False),
        # config 3: the largest, adapters on all four linears of every layer
        dict(name="forward_base_64", kind="forward", model="base", height=224, width=224, frames=64, adapters=3, first=0, sum=False),
        # a layer of the small backbone on its own, a handful of blocks
        dict(name="linear_9", kind="linear", blocks=9, tokens=197, k=192, n=576, rank=8, per_block=2, stack=16, fp32=False),
        # config 5: the isolated multi-adapter linear
        dict(name="linear_256", kind="linear", blocks=256, tokens=197, k=768, n=2304, rank=16, per_block=2, stack=64, fp32=False),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _size(rng):
    """Frame sizes in patches of 16: the square ones of the configurations and camera-shaped ones, at most 197 tokens."""
    return rng.choice([(64, 64), (112, 112), (128, 224), (160, 160), (144, 192), (224, 224), (224, 224), (224, 224)])


def draw(rng):
    """One more case of the same kinds; sizes spread over the whole range, odd ones among them."""
    kind = rng.choice(["select", "stream", "forward", "forward", "forward", "linear", "linear"])
    if kind == "select":
        return dict(kind=kind, frames=_log(rng, 1, 1024), overlap=rng.random() < 0.5, copy=rng.random() < 0.5)
    if kind == "stream":
        h, w = _size(rng)
        return dict(kind=kind, model=rng.choice(["tiny", "preset"]), height=h, width=w, frames=_log(rng, 1, 128), active=rng.randint(1, 3))
    if kind == "linear":
        fp32 = rng.random() < 0.2
        k = rng.choice([192, 384, 768])
        return dict(kind=kind, blocks=_log(rng, 1, 32 if fp32 else 256), tokens=rng.choice([17, 50, 101, 113, 197, 197]), k=k,
                    n=rng.choice([k, 3 * k, 4 * k]) if k < 768 else rng.choice([k, 3 * k]), rank=rng.choice([4, 8, 16, 32]),
                    per_block=rng.randint(1, 3) if k < 768 else rng.randint(1, 2), stack=rng.choice([4, 16, 64]), fp32=fp32)
    model = rng.choice(["fp32", "tiny", "tiny", "preset", "base"])
    h, w = _size(rng)
    most = {"fp32": 64, "tiny": 333, "preset": 333, "base": 60}[model]
    return dict(kind=kind, model=model, height=h, width=w, frames=_log(rng, 1, most), adapters=rng.randint(1, 3),
                first=10 if model == "preset" else 0 if model == "fp32" else rng.choice([0, 10]),
                sum=model in ("tiny", "preset") and rng.random() < 0.3)


# ----------------------------------------------------------------------------- models and contexts

def _cfg(model, height, width):
    base = {"fp32": synth.CFG1, "tiny": synth.CFG2, "base": synth.CFG3,
            "preset": replace(synth.CFG2, name="preset", n_adapters=11, r=32, targets=synth.TGT_QKV, L0=10, lora_scale=2.0)}[model]
    return replace(base, H=height, W=width)


@functools.lru_cache(maxsize=4)
def _weights(model):
    cfg = _cfg(model, 224, 224)
    w = synth.make_weights(cfg, np.random.default_rng(4242))
    if model == "preset":      # query ranks write query columns, value ranks write value columns
        half, d, b = cfg.r // 2, cfg.D, w["B_qkv"]
        b[:, :, :half, d:] = 0.0
        b[:, :, half:, :2 * d] = 0.0
    return w


@functools.lru_cache(maxsize=6)
def _model(model, height, width, first, summed):
    cfg = _cfg(model, height, width)
    w = dict(_weights(model))
    w["pos"] = w["pos"][:cfg.T]
    return binding.DeviceModel(cfg, w, L0=first, compose="sum" if summed else "branch")


@functools.lru_cache(maxsize=1)
def _overlapping():
    """Overlapping contexts over 80 labels, built by the library from co-occurrence counts, and an accuracy table."""
    cooc, _, _ = synth.make_cooccurrence(CONTEXTS, GROUP, n_images=6000, p_partner=0.5, seed=2003, shuffle=False)
    member, _ = binding.poly_build_contexts(cooc, GROUP, 45, allow_overlap=True)
    return member, synth.make_accuracy_table(member)


def _up(a, dtype):
    return torch.from_numpy(np.ascontiguousarray(a)).to(device=DEV, dtype=dtype).contiguous()


def _ints(n):
    return torch.zeros(n, dtype=torch.int32, device=DEV)


def _frames(cfg, count, seed):
    gen = torch.Generator(device=DEV).manual_seed(seed)
    x = torch.rand((count, cfg.H, cfg.W, 3), generator=gen, device=DEV)
    return x.to(torch.bfloat16 if cfg.dtype == synth.DT_BF16 else torch.float32)


def _sets(rng, frames, stack, most):
    """1 + Binomial(most - 1, 0.4) adapters per frame, ascending in a frame."""
    counts = 1 + rng.binomial(most - 1, 0.4, size=frames) if most > 1 else np.ones(frames, dtype=np.int64)
    return [np.sort(rng.choice(stack, size=int(c), replace=False)) for c in counts]


# ----------------------------------------------------------------------------- what a program has in hand before the call

def _prepare_select(case, seed):
    frames = case["frames"]
    scores, _ = synth.make_label_stream(frames, CONTEXTS, GROUP, seed=seed)
    k = scores.shape[1]
    s = dict(kind="select", scores=_up(scores, torch.float32), off=_ints(frames + 1), ids=_ints(8 * frames), cnt=_ints(2),
             state=torch.zeros(binding.poly_select_state_bytes(k), dtype=torch.uint8, device=DEV), copy=case["copy"], acc=None, tau=0.0)
    if case["overlap"]:
        member, acc = _overlapping()
        s.update(member=_up(member, torch.uint8), acc=_up(acc, torch.float32), tau=0.3)
    else:
        s.update(member=_up(synth.make_group_membership(CONTEXTS, GROUP), torch.uint8))
    return s


def _prepare_stream(case, seed):
    model = _model(case["model"], case["height"], case["width"], 10, False)
    cfg, frames = model.cfg, case["frames"]
    rng = np.random.default_rng(seed)
    contexts = cfg.n_adapters
    k = contexts * GROUP
    cap = 4 * frames
    # a confident base head: the labels of `active` contexts are on, all others off, with a spread from the class token
    bias = rng.normal(-6.0, 0.5, size=k).astype(np.float32)
    for c in rng.choice(contexts, size=case["active"], replace=False):
        bias[c * GROUP + rng.choice(GROUP, size=rng.integers(1, 3), replace=False)] = 6.0
    weight = rng.standard_normal((cfg.D, k), dtype=np.float32) / np.float32(np.sqrt(cfg.D))
    head = binding.DeviceStream(model, synth.round_to_bf16(weight), synth.round_to_bf16(bias), synth.make_group_membership(contexts, GROUP))
    ws = torch.empty(binding.poly_stream_step_workspace_bytes(model, frames, cap, k), dtype=torch.uint8, device=DEV)
    return dict(kind="stream", model=model, head=head, frames=_frames(cfg, frames, seed), cap=cap, off=_ints(frames + 1), ids=_ints(cap),
                cnt=_ints(2), status=_ints(1), scores=torch.zeros(cap, cfg.C, device=DEV), logits=torch.zeros(cap, cfg.C, device=DEV),
                base=torch.zeros(frames, k, device=DEV), merged=torch.zeros(frames, k, device=DEV), ws=ws)


def _prepare_forward(case, seed):
    model = _model(case["model"], case["height"], case["width"], case["first"], case["sum"])
    cfg, frames, most = model.cfg, case["frames"], case["adapters"]
    rng = np.random.default_rng(seed)
    k = cfg.n_adapters * cfg.C
    cap = most * frames
    # scores of a monitor that sees one or two labels of every context in a frame's set
    label = rng.uniform(0.0, 0.4, size=(frames, k)).astype(np.float32)
    for f, ids in enumerate(_sets(rng, frames, cfg.n_adapters, most)):
        for c in ids:
            label[f, c * cfg.C + rng.integers(0, cfg.C, size=2)] = rng.uniform(0.6, 1.0)
    ws = torch.empty(binding.poly_forward_workspace_bytes(model, frames, cap), dtype=torch.uint8, device=DEV)
    return dict(kind="forward", model=model, label=_up(label, torch.float32), frames=_frames(cfg, frames, seed), cap=cap,
                member=_up(synth.make_group_membership(cfg.n_adapters, cfg.C), torch.uint8), off=_ints(frames + 1), ids=_ints(cap),
                cnt=_ints(2), status=_ints(1), scores=torch.zeros(cap, cfg.C, device=DEV), logits=torch.zeros(cap, cfg.C, device=DEV),
                merged=torch.zeros(frames, k, device=DEV), ws=ws)


def _prepare_linear(case, seed):
    b, t, k, n, r, stack = (case[x] for x in ("blocks", "tokens", "k", "n", "rank", "stack"))
    gen = torch.Generator(device=DEV).manual_seed(seed)
    elt = torch.float32 if case["fp32"] else torch.bfloat16
    norm = lambda shape, std: (torch.randn(shape, generator=gen, device=DEV) * std)  # noqa: E731
    rng = np.random.default_rng(seed)
    sets = [sorted(rng.choice(stack, size=min(case["per_block"], stack), replace=False)) for _ in range(b)]
    off, ids = synth.sets_to_csr(sets)
    rows = int(off[-1])
    ws = torch.empty(binding.poly_lora_linear_workspace_bytes(b, t, r, rows, int(not case["fp32"])), dtype=torch.uint8, device=DEV)
    return dict(kind="linear", x=norm((b, t, k), 1.0).to(elt), w=norm((n, k), 0.02).to(elt), bias=norm((n,), 0.02),
                at=norm((stack, r, k), 1.0 / r).to(elt), bt=norm((stack, n, r), 0.02).to(elt), off=_up(off, torch.int32),
                ids=_up(ids, torch.int32), rows=rows, y=torch.zeros((rows, t, n), dtype=elt, device=DEV), status=_ints(1), ws=ws)


def prepare(case, seed):
    return {"select": _prepare_select, "stream": _prepare_stream, "forward": _prepare_forward, "linear": _prepare_linear}[case["kind"]](case, seed)


def run(s):
    """One pass through the entry points; the outputs are the caller's own buffers."""
    if s["kind"] == "select":
        binding.poly_select(s["scores"], s["member"], s["off"], s["ids"], s["cnt"], context_copy=s["copy"], acc=s["acc"], tau=s["tau"],
                            state=s["state"])
        return [s["off"], s["ids"], s["cnt"], s["state"]]
    if s["kind"] == "stream":
        binding.poly_stream_step(s["model"], s["head"], s["frames"], s["cap"], s["off"], s["ids"], s["cnt"], s["scores"], s["ws"],
                                 out_base_scores=s["base"], out_logits=s["logits"], out_merged=s["merged"], dev_status=s["status"])
        return [s["off"], s["ids"], s["cnt"], s["status"], s["base"], s["logits"], s["scores"], s["merged"], s["head"].state, s["head"].carry]
    if s["kind"] == "forward":
        binding.poly_select(s["label"], s["member"], s["off"], s["ids"], s["cnt"])
        binding.poly_forward(s["model"], s["frames"], s["off"], s["ids"], s["cap"], s["scores"], s["ws"], out_logits=s["logits"],
                             out_merged=s["merged"], dev_status=s["status"])
        return [s["off"], s["ids"], s["cnt"], s["status"], s["logits"], s["scores"], s["merged"]]
    binding.poly_lora_linear(s["x"], s["w"], s["bias"], s["at"], s["bt"], 1.0, s["off"], s["ids"], s["rows"], s["y"], s["ws"],
                             dev_status=s["status"])
    return [s["y"], s["status"]]


# ----------------------------------------------------------------------------- what a pass cannot do without

def _layer_flops(cfg):
    """Base linears and attention of one layer on one token block."""
    return 2.0 * cfg.T * (4 * cfg.D * cfg.D + 2 * cfg.D * cfg.Dm) + 4.0 * cfg.T * cfg.T * cfg.D


def _lora_flops(cfg):
    return sum(2.0 * cfg.T * cfg.r * (i + o) for i, o in cfg.target_dims().values())


def _model_work(cfg, frames, rows, first, summed):
    """rows = (frame, adapter) pairs.  Weights once, the adapters in use once, frames in, scores out."""
    es = 2 if cfg.dtype == synth.DT_BF16 else 4
    adapted = cfg.L - first
    flops = 2.0 * frames * (cfg.T - 1) * cfg.patch_dim * cfg.D + frames * first * _layer_flops(cfg)
    flops += adapted * ((frames if summed else rows) * _layer_flops(cfg) + rows * _lora_flops(cfg))
    if not summed and adapted:   # the base product of the first adapted qkv linear is shared by a frame's branches
        flops -= (rows - frames) * 2.0 * cfg.T * cfg.D * 3 * cfg.D
    flops += rows * 2.0 * cfg.D * cfg.C
    weights = cfg.patch_dim * cfg.D + cfg.L * (4 * cfg.D * cfg.D + 2 * cfg.D * cfg.Dm) + cfg.T * cfg.D
    used = cfg.n_adapters * (1.0 - (1.0 - 1.0 / cfg.n_adapters) ** rows)
    adapters = used * (adapted * sum(cfg.r * (i + o) for i, o in cfg.target_dims().values()) + cfg.C * cfg.D)
    k = cfg.n_adapters * cfg.C
    return {"bytes": es * (frames * cfg.H * cfg.W * 3 + weights + adapters) + 4.0 * (2 * rows * cfg.C + 2 * frames * k), "flops": flops}


def work(case):
    if case["kind"] == "select":
        k = CONTEXTS * GROUP
        table = 45 * k * 5 if case["overlap"] else CONTEXTS * k
        return {"bytes": 4.0 * case["frames"] * k + table + 4.0 * (case["frames"] + 1) + 4.0 * 2.5 * case["frames"], "flops": 0.0}
    if case["kind"] == "stream":
        cfg = _cfg(case["model"], case["height"], case["width"])
        w = _model_work(cfg, case["frames"], case["active"] * case["frames"], 10, False)
        k = cfg.n_adapters * GROUP
        return {"bytes": w["bytes"] + 2.0 * cfg.D * k + 4.0 * case["frames"] * k, "flops": w["flops"] + 2.0 * case["frames"] * cfg.D * k}
    if case["kind"] == "forward":
        cfg = _cfg(case["model"], case["height"], case["width"])
        return _model_work(cfg, case["frames"], case["frames"] * (1.0 + 0.4 * (case["adapters"] - 1)), case["first"], case["sum"])
    b, t, k, n, r, stack = (case[x] for x in ("blocks", "tokens", "k", "n", "rank", "stack"))
    es, per = 4 if case["fp32"] else 2, min(case["per_block"], stack)
    rows = b * per
    used = stack * (1.0 - (1.0 - per / stack) ** b)
    return {"bytes": es * (b * t * k + n * k + used * r * (k + n) + rows * t * n) + 4.0 * n,
            "flops": 2.0 * b * t * k * n + 2.0 * rows * t * r * (k + n)}


def tolerance(case):
    """Selections are whole numbers.  Products in bf16 round every activation to 8 bits; in fp32 only the order of the sums differs."""
    if case["kind"] == "select":
        return "exact"
    if case.get("fp32") or case.get("model") == "fp32":
        return {"rel": 1e-5}
    return {"rel": 1e-2}
