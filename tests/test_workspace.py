"""Sizes of the forward's workspace: a workspace for the largest call of a program serves its smaller ones (no GPU needed)."""
import ctypes as C
from dataclasses import replace

import pytest

from paper_2507_14959_amd import binding, synth


def _desc(cfg, L0, compose=0):
    return binding.ModelDesc(cfg.H, cfg.W, cfg.patch, cfg.D, cfg.heads, cfg.L, cfg.Dm, L0, cfg.targets, cfg.r, cfg.n_adapters, cfg.C,
                             cfg.dtype, 1.0, 1e-6, compose)


@pytest.mark.parametrize("name,cfg,L0,compose", [
    ("branch", synth.CFG2, 0, 0),
    ("branch, shared trunk", synth.CFG2, 10, 0),
    ("sum", synth.CFG2, 0, 1),
    ("sum, shared trunk", replace(synth.CFG2, targets=15), 9, 1),
    ("short blocks", replace(synth.CFG2, H=64, W=64), 5, 0),
    ("nine layers", replace(synth.CFG2, L=9), 0, 0),
    ("no adapted layer", synth.CFG2, 12, 0),
    ("fp32", synth.CFG1, 0, 0),
    ("wide", synth.CFG3, 0, 0),
])
def test_workspace_never_shrinks_with_frames_or_row_blocks(name, cfg, L0, compose):
    d = _desc(cfg, L0, compose)
    lib = binding.lib()
    for size in (lib.poly_forward_workspace_bytes, lambda m, F, R: lib.poly_stream_step_workspace_bytes(m, F, R, 80)):
        at = {(F, R): size(C.byref(d), F, R) for F in range(1, 72) for R in list(range(0, 72)) + [96, 160, 400]}
        for (F, R), b in at.items():
            assert b > 0
            for more in ((F + 1, R), (F, R + 1), (F, 400)):
                assert more not in at or at[more] >= b, (F, R, more, b, at[more])


def test_the_tasks_of_few_blocks_do_not_multiply_the_workspace():
    """Per-layer buffers are bounded: DeiT-tiny with adapters on every layer, against the row kernels' own 2.8 MB per 1 frame and 3 row-blocks."""
    d = _desc(synth.CFG2, 0)
    f = binding.lib().poly_forward_workspace_bytes
    mib = lambda F, R: f(C.byref(d), F, R) / 2 ** 20          # noqa: E731
    assert mib(1, 3) < 40 and mib(6, 20) < 140 and mib(32, 96) < 155
