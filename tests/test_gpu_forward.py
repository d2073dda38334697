"""poly_forward on the GPU against the CPU checker.

Tolerances (max-abs on logits): 1e-4 in fp32, 2e-2 in bf16 -- the checker is the exact result on the
same bf16-valued parameters; the GPU rounds activations to bf16 between stages and accumulates in fp32.
"""
import dataclasses
import functools

import numpy as np
import pytest
import torch

import oracle
from paper_2507_14959_amd import binding, synth

pytestmark = pytest.mark.gpu

TOL = {synth.DT_F32: 1e-4, synth.DT_BF16: 2e-2}


def compare(cfg, w, frames, off, ids, L0, K=0, compose="branch", tol=None):
    tol = tol or TOL[cfg.dtype]
    model = binding.DeviceModel(cfg, w, L0=L0, compose=compose)
    got = binding.run_forward(model, frames, off, ids, K=K)
    want = oracle.forward(cfg, w, frames, off, ids, L0=L0, K=K, compose=compose)
    assert got["status"] == 0
    err = np.abs(got["logits"] - want["logits"]).max() if off[-1] else 0.0
    assert err < tol, f"logits max-abs error {err}"
    if off[-1]:
        assert np.abs(got["scores"] - want["scores"]).max() < tol
    if K:
        assert np.abs(got["merged"] - want["merged"]).max() < tol
    return got, want, err


@pytest.mark.parametrize("L0", [0, 1, 2])
def test_config1_fp32(L0):
    cfg, w, frames, off, ids = synth.make_forward_case(1)
    compare(cfg, w, frames, off, ids, L0, K=cfg.n_adapters * cfg.C)


@pytest.mark.parametrize("dtype", [synth.DT_F32, synth.DT_BF16])
@pytest.mark.parametrize("targets,L0,r", [(15, 0, 4), (3, 1, 8), (12, 0, 16), (5, 3, 4), (10, 2, 20)])
def test_small_models_all_target_sets(dtype, targets, L0, r):
    cfg, w, frames, off, ids = synth.make_small_case(40 + targets, dtype=dtype, targets=targets, L=3, F=5, r=r, max_set=3,
                                                      n_adapters=4, hw=48, patch=8)   # T = 37: ragged in every tile
    compare(cfg, w, frames, off, ids, L0, K=cfg.n_adapters * cfg.C)


@pytest.mark.parametrize("D,heads,Dm,hw,r,targets,L0", [
    (64, 1, 128, 48, 4, 3, 0),      # one 64-column tile, T = 37: a single ragged row tile
    (64, 1, 192, 64, 16, 1, 1),     # T = 65: a full tile and a one-row tile; adapters on qkv only; fan-out at layer 1
    (128, 2, 256, 64, 12, 3, 0),    # rank 12: the second half of the expand operand is partly empty
    (192, 3, 768, 40, 8, 3, 2),     # DeiT-tiny widths, T = 26, fan-out at layer 2
    (192, 3, 320, 72, 16, 2, 0),    # adapters on proj only, Dm = 5 chunks, T = 82
    (128, 2, 384, 64, 8, 3, 0),     # Dm = 6 chunks: the last feed-forward item and the second qkv item share a stage of the weight ring
])
def test_row_kernels_all_widths(D, heads, Dm, hw, r, targets, L0):
    """bf16 models that the fused row kernels take (no adapters on fc1 / fc2): every tile width, ragged tiles.  (So few blocks run as tasks;
    test_gpu_layer_kernels.py has the row kernels on the same cases.)"""
    cfg, w, frames, off, ids = synth.make_small_case(60 + D + r, dtype=synth.DT_BF16, targets=targets, L=4, F=4, r=r, max_set=3,
                                                      n_adapters=5, D=D, heads=heads, Dm=Dm, hw=hw, patch=8)
    compare(cfg, w, frames, off, ids, L0, K=cfg.n_adapters * cfg.C)


@pytest.mark.parametrize("D,heads,Dm,hw,r,targets,L0", [
    (256, 4, 512, 40, 8, 15, 0),    # LayerNorm rows of one 16-byte piece per lane; shrink over K = 256 and 512
    (512, 8, 1024, 48, 16, 15, 1),  # two pieces per lane; T = 37
    (320, 5, 640, 40, 4, 15, 0),    # D not a multiple of 256: the strided LayerNorm; shrink with 20 and 40 K steps (5 and 10 per wave)
    (256, 4, 1024, 72, 16, 3, 0),   # adapters on qkv and proj only: the layer splits into GEMM kernels without the feed-forward shrink
])
def test_wide_path_widths(D, heads, Dm, hw, r, targets, L0):
    """bf16 models wider than the fused row kernels: LayerNorm, shrink, GEMM and attention kernels at other widths than ViT-base's."""
    cfg, w, frames, off, ids = synth.make_small_case(90 + D + r, dtype=synth.DT_BF16, targets=targets, L=2, F=5, r=r, max_set=3,
                                                      n_adapters=4, D=D, heads=heads, Dm=Dm, hw=hw, patch=8)
    compare(cfg, w, frames, off, ids, L0, K=cfg.n_adapters * cfg.C)


@pytest.mark.parametrize("D,heads,Dm,hw,r,targets,L0", [(64, 1, 192, 64, 16, 1, 1), (128, 2, 384, 64, 8, 3, 0), (192, 3, 768, 40, 8, 3, 2)])
def test_row_kernels_repeat_bitwise(D, heads, Dm, hw, r, targets, L0):
    """The fused row kernels hand LDS stages from a stream wave to the computing waves by hand-counted waits: a stage that is
    refilled one step early shows up as run-to-run differences long before it shows up as a wrong answer.  (So few blocks run as tasks, with
    the same symptom for a task that starts early; test_gpu_layer_kernels.py repeats the row kernels.)"""
    cfg, w, frames, off, ids = synth.make_small_case(60 + D + r, dtype=synth.DT_BF16, targets=targets, L=4, F=4, r=r, max_set=3,
                                                      n_adapters=5, D=D, heads=heads, Dm=Dm, hw=hw, patch=8)
    model = binding.DeviceModel(cfg, w, L0=L0)
    first = binding.run_forward(model, frames, off, ids)["logits"]
    for _ in range(8):
        again = binding.run_forward(model, frames, off, ids)["logits"]
        assert np.array_equal(first, again)


@pytest.mark.parametrize("D,heads,Dm,hw,r,targets,L0,F", [
    (64, 1, 128, 48, 4, 3, 0, 75),      # the cases of test_row_kernels_all_widths on so many blocks that they leave the task queue
    (64, 1, 192, 64, 16, 1, 1, 50),
    (128, 2, 384, 64, 12, 3, 0, 50),
    (192, 3, 768, 40, 8, 3, 2, 145),
    (192, 3, 320, 72, 16, 2, 0, 50),
])
def test_row_kernels_on_many_blocks(D, heads, Dm, hw, r, targets, L0, F):
    cfg, w, frames, off, ids = synth.make_small_case(60 + D + r, dtype=synth.DT_BF16, targets=targets, L=3, F=F, r=r, max_set=3,
                                                      n_adapters=5, D=D, heads=heads, Dm=Dm, hw=hw, patch=8)
    compare(cfg, w, frames, off, ids, L0, K=cfg.n_adapters * cfg.C)
    model = binding.DeviceModel(cfg, w, L0=L0)
    first = binding.run_forward(model, frames, off, ids)["logits"]
    assert np.array_equal(first, binding.run_forward(model, frames, off, ids)["logits"])


@pytest.mark.parametrize("compose", ["branch", "sum"])
@pytest.mark.parametrize("D,heads,Dm,hw,r,targets,L0,F", [
    (64, 1, 128, 16, 4, 15, 0, 1),      # T = 5: one ragged row tile, one K step per half; a single block
    (64, 1, 256, 64, 32, 15, 1, 5),     # T = 65: a one-row tile; two full rank tiles; coarse tasks
    (128, 2, 256, 40, 20, 15, 0, 9),    # rank 20: the second rank tile partly empty; more blocks than queues
    (192, 3, 768, 112, 8, 3, 1, 2),     # DeiT-tiny widths and tokens
    (192, 3, 640, 24, 12, 15, 2, 4),    # Dm no multiple of 256: no coarse tasks
    (192, 3, 768, 32, 4, 15, 0, 100),   # T = 17, many blocks per queue
])
def test_task_queue_sizes(D, heads, Dm, hw, r, targets, L0, F, compose):
    """Layers as tasks of 32 rows: tile edges, rank tiles, one block to many per queue; repeated bitwise (a task that starts before
    its inputs are complete shows up as run-to-run differences)."""
    cfg, w, frames, off, ids = synth.make_small_case(300 + D + r, dtype=synth.DT_BF16, targets=targets, L=3, F=F, r=r, max_set=3,
                                                      n_adapters=5, D=D, heads=heads, Dm=Dm, hw=hw, patch=8)
    model = binding.DeviceModel(cfg, w, L0=L0, compose=compose)
    got = binding.run_forward(model, frames, off, ids)
    want = oracle.forward(cfg, w, frames, off, ids, L0=L0, compose=compose)
    assert got["status"] == 0
    if len(ids):
        assert np.abs(got["logits"] - want["logits"]).max() < TOL[cfg.dtype]
    for _ in range(5):
        assert np.array_equal(got["logits"], binding.run_forward(model, frames, off, ids)["logits"])


def test_frames_without_adapters_and_empty_batch():
    cfg, w, frames, _, _ = synth.make_small_case(50, dtype=synth.DT_BF16, F=4)
    off, ids = synth.sets_to_csr([[], [1, 0], [], [2]])
    got, want, _ = compare(cfg, w, frames, off, ids, 0, K=cfg.n_adapters * cfg.C)
    assert np.array_equal(got["merged"][0], np.zeros(cfg.n_adapters * cfg.C))
    off, ids = synth.sets_to_csr([[], [], [], []])
    model = binding.DeviceModel(cfg, w)
    got = binding.run_forward(model, frames, off, ids, K=cfg.n_adapters * cfg.C)
    assert got["status"] == 0 and np.array_equal(got["merged"], np.zeros((4, cfg.n_adapters * cfg.C)))


def test_row_bound_above_R_and_bad_ids():
    cfg, w, frames, off, ids = synth.make_small_case(51, dtype=synth.DT_BF16, F=4, max_set=2)
    model = binding.DeviceModel(cfg, w)
    a = binding.run_forward(model, frames, off, ids)
    b = binding.run_forward(model, frames, off, ids, R_cap=int(off[-1]) + 5)
    R = int(off[-1])
    assert np.array_equal(a["logits"], b["logits"][:R]) and np.all(np.isnan(b["logits"][R:]))
    bad = ids.copy(); bad[0] = cfg.n_adapters
    c = binding.run_forward(model, frames, off, bad)
    assert c["status"] == binding.POLY_ERANGE and np.all(np.isnan(c["logits"]))


def test_position_invariance_is_bitwise_and_zero_B_is_bare_backbone():
    cfg, w, frames, _, _ = synth.make_small_case(52, dtype=synth.DT_BF16, F=2, n_adapters=4)
    fr = np.stack([frames[0], frames[1], frames[0], frames[0]])
    off, ids = synth.sets_to_csr([[0, 2], [1], [2], [3, 2, 0]])
    model = binding.DeviceModel(cfg, w)
    out = binding.run_forward(model, fr, off, ids)["logits"]
    assert np.array_equal(out[1], out[3]) and np.array_equal(out[1], out[5]) and np.array_equal(out[0], out[6])
    wz = {k: (np.zeros_like(v) if k.startswith("B_") else v) for k, v in w.items()}
    z = binding.run_forward(binding.DeviceModel(cfg, wz), fr, off, ids)["logits"]
    bare = binding.run_forward(binding.DeviceModel(cfg, w, L0=cfg.L), fr, off, ids)["logits"]
    # Adapters on all four linears send the MLP half through other kernels than the bare backbone takes (the
    # fused MLP kernel has no low-rank branch): same mathematics, other summation order, so only close.
    assert np.abs(z - bare).max() < 5e-3
    # Adapters on qkv and proj only: every layer runs the same kernels with or without the adapters, and a zero
    # B adds exact zeros to the accumulators.
    cfg2 = dataclasses.replace(cfg, targets=synth.TGT_QKV | synth.TGT_PROJ)
    z2 = binding.run_forward(binding.DeviceModel(cfg2, wz), fr, off, ids)["logits"]
    bare2 = binding.run_forward(binding.DeviceModel(cfg2, w, L0=cfg.L), fr, off, ids)["logits"]
    assert np.abs(z2 - bare2).max() < 1e-6 and np.abs(bare2 - bare).max() < 1e-6


@pytest.mark.parametrize("L0", [0, 10])
def test_config2_deit_tiny_full(L0):
    cfg, w, frames, off, ids = synth.make_forward_case(2)
    _, _, err = compare(cfg, w, frames, off, ids, L0, K=cfg.n_adapters * cfg.C)
    print(f"config 2, L0={L0}: R={off[-1]}, logits max-abs error {err:.2e}")


@functools.lru_cache(maxsize=1)
def _config3_on_gpu():
    cfg, w, frames, off, ids = synth.make_forward_case(3)
    got = binding.run_forward(binding.DeviceModel(cfg, w), frames, off, ids)     # the full 64-frame launch, 133 row-blocks
    return cfg, w, frames, off, ids, got


@pytest.mark.parametrize("part", range(4))
def test_config3_vit_base_full_size_every_frame(part):
    """Every row-block of the full-size launch against the checker, 16 frames per test (the checker needs about 12 core-seconds
    per row-block)."""
    cfg, w, frames, off, ids, got = _config3_on_gpu()
    assert got["status"] == 0 and got["logits"].shape == (int(off[-1]), cfg.C)
    f0, f1 = 16 * part, 16 * (part + 1)
    o1, i1 = synth.sets_to_csr([list(ids[off[f]:off[f + 1]]) for f in range(f0, f1)])
    want = oracle.forward(cfg, w, frames[f0:f1], o1, i1)
    err = np.abs(got["logits"][off[f0]:off[f1]] - want["logits"]).max()
    print(f"config 3 frames {f0}..{f1 - 1} ({len(i1)} row-blocks): logits max-abs error {err:.2e}")
    assert err < TOL[synth.DT_BF16]
    assert np.abs(got["scores"][off[f0]:off[f1]] - want["scores"]).max() < TOL[synth.DT_BF16]


def test_config4_select_then_forward_without_host_round_trip():
    """All 16 batches of the 1024-frame stream: poly_select feeds poly_forward on the device; the adapter sets of every frame are
    compared bit for bit, the logits on four frames of every batch (the frames differ from batch to batch)."""
    cfg = synth.CFG4
    rng = np.random.default_rng(synth.seed_of(4))
    w = synth.make_weights(cfg, rng)
    mem = synth.make_group_membership()
    scores, _ = synth.make_label_stream(1024)
    model = binding.DeviceModel(cfg, w)
    dev = "cuda"
    cap = 64 * 5
    ws = torch.empty(binding.poly_forward_workspace_bytes(model, 64, cap), dtype=torch.uint8, device=dev)
    m = torch.from_numpy(mem).to(dev)
    worst = 0.0
    for batch in range(16):
        frames = synth.make_frames(cfg, 64, np.random.default_rng([synth.seed_of(4), batch]))
        s = torch.from_numpy(scores[batch * 64:(batch + 1) * 64]).to(dev)
        off = torch.zeros(65, dtype=torch.int32, device=dev); ids = torch.zeros(cap, dtype=torch.int32, device=dev)
        cnt = torch.zeros(2, dtype=torch.int32, device=dev); st = torch.zeros(1, dtype=torch.int32, device=dev)
        out = torch.full((cap, cfg.C), float("nan"), device=dev); lg = torch.full((cap, cfg.C), float("nan"), device=dev)
        binding.poly_select(s, m, off, ids, cnt)
        binding.poly_forward(model, model.frames_to_device(frames), off, ids, cap, out, ws, out_logits=lg, dev_status=st)
        torch.cuda.synchronize()
        o_off, o_ids, _ = oracle.select(scores[batch * 64:(batch + 1) * 64], mem)
        assert np.array_equal(off.cpu().numpy(), o_off) and np.array_equal(ids.cpu().numpy()[:len(o_ids)], o_ids)
        R = len(o_ids)
        sub = sorted({0, 63, (7 * batch + 3) % 64, (11 * batch + 29) % 64})     # frames the checker recomputes
        o1, i1 = synth.sets_to_csr([list(o_ids[o_off[f]:o_off[f + 1]]) for f in sub])
        want = oracle.forward(cfg, w, frames[sub], o1, i1)
        g = np.concatenate([lg.cpu().numpy()[o_off[f]:o_off[f + 1]] for f in sub])
        if len(i1):
            worst = max(worst, float(np.abs(g - want["logits"]).max()))
        assert worst < TOL[synth.DT_BF16], (batch, worst)
        assert int(st.item()) == 0 and np.all(np.isnan(lg.cpu().numpy()[R:])) and np.isfinite(lg.cpu().numpy()[:R]).all()
    print(f"config 4: logits max-abs error over 16 batches {worst:.2e}")


@pytest.mark.parametrize("D,heads,Dm,hw,r,targets,L0,dtype", [
    (192, 3, 768, 40, 8, 3, 1, synth.DT_BF16),      # narrow (few blocks: as tasks; row kernels in test_gpu_layer_kernels.py)
    (256, 4, 512, 40, 16, 15, 0, synth.DT_BF16),    # shrink kernel + expand in the GEMM
    (128, 2, 256, 32, 4, 15, 0, synth.DT_F32),
])
def test_lora_scale_and_layernorm_eps_other_than_the_defaults(D, heads, Dm, hw, r, targets, L0, dtype):
    """The paper's adapters are trained with a scaling factor of 32 at rank 16 (Sec. 4), i.e. s = 2."""
    cfg, w, frames, off, ids = synth.make_small_case(130 + D, dtype=dtype, targets=targets, L=3, F=4, r=r, max_set=3, n_adapters=4, D=D,
                                                      heads=heads, Dm=Dm, hw=hw, patch=8)
    cfg = dataclasses.replace(cfg, lora_scale=2.0, ln_eps=1e-5)
    _, want, _ = compare(cfg, w, frames, off, ids, L0, K=cfg.n_adapters * cfg.C)
    plain = oracle.forward(dataclasses.replace(cfg, lora_scale=1.0), w, frames, off, ids, L0=L0)
    assert np.abs(plain["logits"] - want["logits"]).max() > 4 * TOL[dtype]        # the scale is visible at this tolerance


def test_rank_outside_the_row_layer_kernel_takes_the_single_linear_and_mlp_kernels():
    """Adapters on qkv and proj with rank 20 at D = 192: the one-launch-per-layer kernel refuses the rank, so proj runs as a GEMM
    with the shrink kernel and the MLP half in the fused MLP kernel.  (Not for so few blocks, which run as tasks: the kernels named here run
    in the test of the same case in test_gpu_layer_kernels.py.)"""
    cfg, w, frames, off, ids = synth.make_small_case(140, dtype=synth.DT_BF16, targets=3, L=3, F=5, r=20, max_set=3, n_adapters=4,
                                                      D=192, heads=3, Dm=768, hw=72, patch=8)     # T = 82: a full and a ragged tile
    compare(cfg, w, frames, off, ids, 0, K=cfg.n_adapters * cfg.C)
    compare(cfg, w, frames, off, ids, 2, K=cfg.n_adapters * cfg.C)


# ------------------------------------------------- several adapters summed on one hidden state per frame (Sec. 3.1)

@pytest.mark.parametrize("dtype", [synth.DT_F32, synth.DT_BF16])
@pytest.mark.parametrize("targets,L0,r", [(15, 0, 4), (3, 1, 8), (12, 0, 16), (5, 2, 4), (10, 3, 20)])
def test_sum_composition_small_models_all_target_sets(dtype, targets, L0, r):
    cfg, w, frames, _, _ = synth.make_small_case(240 + targets, dtype=dtype, targets=targets, L=3, F=5, r=r, max_set=3,
                                                  n_adapters=4, hw=48, patch=8)   # T = 37; L0 = 3: no adapted layer at all
    off, ids = synth.sets_to_csr([[0, 2, 3], [], [1, 3], [2], [3, 1, 0]])
    _, want, _ = compare(cfg, w, frames, off, ids, L0, K=cfg.n_adapters * cfg.C, compose="sum")
    if L0 < cfg.L:
        branch = oracle.forward(cfg, w, frames, off, ids, L0=L0)
        assert np.abs(branch["logits"] - want["logits"]).max() > 2 * TOL[dtype]     # the two readings differ visibly here


@pytest.mark.parametrize("D,heads,Dm,hw,r,targets,L0", [
    (192, 3, 768, 72, 8, 3, 2),      # DeiT-tiny widths, T = 82 (few blocks: as tasks; by layer in test_gpu_layer_kernels.py)
    (192, 3, 768, 72, 16, 1, 0),     # adapters on qkv only (as above)
    (256, 4, 1024, 72, 16, 15, 1),   # wide path throughout
    (768, 12, 1024, 64, 16, 15, 0),  # ViT-base width: the large GEMM tiles with summed terms
])
def test_sum_composition_bf16_widths(D, heads, Dm, hw, r, targets, L0):
    cfg, w, frames, off, ids = synth.make_small_case(260 + D + r, dtype=synth.DT_BF16, targets=targets, L=4, F=6, r=r, max_set=3,
                                                      n_adapters=5, D=D, heads=heads, Dm=Dm, hw=hw, patch=8)
    compare(cfg, w, frames, off, ids, L0, K=cfg.n_adapters * cfg.C, compose="sum")


def test_sum_composition_one_adapter_per_frame_is_the_branch_result_and_bad_ids_write_nothing():
    cfg, w, frames, _, _ = synth.make_small_case(270, dtype=synth.DT_BF16, F=4, targets=15, n_adapters=4, D=256, heads=4, Dm=512, hw=40, patch=8)
    off, ids = synth.sets_to_csr([[1], [], [3], [0]])
    a = binding.run_forward(binding.DeviceModel(cfg, w), frames, off, ids)
    b = binding.run_forward(binding.DeviceModel(cfg, w, compose="sum"), frames, off, ids)
    assert np.array_equal(a["logits"], b["logits"])      # same kernels, same operands, same order
    bad = ids.copy(); bad[1] = cfg.n_adapters
    c = binding.run_forward(binding.DeviceModel(cfg, w, compose="sum"), frames, off, bad)
    assert c["status"] == binding.POLY_ERANGE and np.all(np.isnan(c["logits"]))


@pytest.mark.parametrize("compose", ["branch", "sum"])
def test_paper_preset_query_value_rank16_scale2_last_two_layers(compose):
    """Sec. 4: rank 16, scaling factor 32 (s = 2), query + value only, adapters on the last 20 % of the layers, 11 contexts."""
    cfg, w, frames, off, ids = synth.make_paper_preset(F=8)
    assert cfg.L0 == cfg.polymorph_L0() == 10 and cfg.lora_scale == 2.0
    _, want, err = compare(cfg, w, frames, off, ids, cfg.L0, K=cfg.n_adapters * cfg.C, compose=compose)
    # the key columns of the qkv adapter are silent: the same weights with only the query and value blocks kept
    print(f"paper preset ({compose}): R={off[-1]}, logits max-abs error {err:.2e}")


@pytest.mark.parametrize("hw,L0", [(48, 1), (88, 0), (128, 1)])
def test_fp32_attention_query_groups_and_key_tiles(hw, L0):
    """fp32 attention at T = 37, 122 and 257 tokens: one to three groups of 128 queries, the last key tile full, cut short and with one key."""
    cfg, w, frames, off, ids = synth.make_small_case(700 + hw, dtype=synth.DT_F32, targets=15, L=2, F=2, r=4, max_set=2, n_adapters=3, hw=hw, patch=8)
    compare(cfg, w, frames, off, ids, L0, K=cfg.n_adapters * cfg.C)
