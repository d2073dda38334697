"""LayerNorm in one launch with the shrink of its rows (wide models, ranks up to 16), or with the product (few rows of the 768-wide one, no adapters)."""
import numpy as np
import pytest

import oracle
from paper_2507_14959_amd import binding, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,hw,F,r,targets,L0,compose", [
    (256, 32, 5, 16, 5, 0, "branch"),        # T = 17: a row in the second tile of 16; frames fan out into three, two, one and no row-blocks
    (512, 16, 6, 4, 15, 1, "branch"),        # T = 5
    (768, 112, 6, 8, 15, 0, "branch"),       # T = 197, more blocks than run as tasks
    (768, 56, 12, 12, 1, 1, "sum"),          # T = 50; all pairs of a frame on its block
    (1024, 48, 4, 16, 4, 0, "sum"),          # T = 37; adapters on fc1 only
])
def test_against_the_oracle(D, hw, F, r, targets, L0, compose):
    cfg, w, frames, _, _ = synth.make_small_case(970 + D + hw, dtype=synth.DT_BF16, targets=targets, L=2, F=F, r=r, n_adapters=5, D=D, heads=D // 64, Dm=512,
                                                 hw=hw, patch=8)
    off, ids = synth.sets_to_csr([[[0, 2, 4], [1, 3], [], [4]][f % 4] for f in range(F)])
    model = binding.DeviceModel(cfg, w, L0=L0, compose=compose)
    binding.poly_profile_begin(200)
    try:
        got = binding.run_forward(model, frames, off, ids)
    finally:
        prof = binding.poly_profile_end()
    alone = (cfg.L - L0) * sum(bool(targets & t) for t in (2, 8))            # proj and fc2
    assert prof["shrink"]["launches"] == alone
    err = np.abs(got["logits"] - oracle.forward(cfg, w, frames, off, ids, L0=L0, compose=compose)["logits"]).max()
    print(f"logits max-abs error {err:.2e}")
    assert got["status"] == 0 and err < 8e-3                                 # (as the layers of test_product_tiles.py)


def test_rejected_arrays_write_nothing():
    cfg, w, frames, _, _ = synth.make_small_case(990, dtype=synth.DT_BF16, targets=5, L=2, F=4, r=8, n_adapters=4, D=256, heads=4, Dm=512, hw=40, patch=8)
    off, ids = synth.sets_to_csr([[1, 2], [], [3], [0]])
    for compose in ("branch", "sum"):
        bad = ids.copy()
        bad[2] = cfg.n_adapters
        got = binding.run_forward(binding.DeviceModel(cfg, w, compose=compose), frames, off, bad)
        assert got["status"] == binding.POLY_ERANGE and np.isnan(got["logits"]).all()


@pytest.mark.parametrize("hw,F,Dm,targets,L0", [
    (112, 2, 520, 3, 2),         # 394 rows: seven tiles, the last of ten rows; 520 columns: the last tile of eight; no adapted layer
    (56, 7, 512, 2, 1),          # T = 50, 350 rows; adapters on proj alone: LayerNorm with the product in the adapted layer too
    (56, 6, 512, 2, 1),          # 300 rows: five tiles, two launches
])
def test_norm_with_the_product_against_the_oracle(hw, F, Dm, targets, L0):
    cfg, w, frames, _, _ = synth.make_small_case(1000 + hw + F, dtype=synth.DT_BF16, targets=targets, L=2, F=F, r=20, n_adapters=3, D=768, heads=12, Dm=Dm, hw=hw, patch=8)
    off, ids = synth.sets_to_csr([[f % 3] for f in range(F)])
    model = binding.DeviceModel(cfg, w, L0=L0)
    binding.poly_profile_begin(200)
    try:
        got = binding.run_forward(model, frames, off, ids)
    finally:
        prof = binding.poly_profile_end()
    again = binding.run_forward(model, frames, off, ids)
    want = oracle.forward(cfg, w, frames, off, ids, L0=L0)["logits"]
    err = np.abs(got["logits"] - want).max()
    print(f"logits max-abs error {err:.2e}")
    # (the layer in which frames fan out has LayerNorm1 and its product in two launches)
    assert prof["layernorm"]["launches"] == (4 if F == 6 else 1 if L0 < cfg.L else 0)
    assert got["status"] == 0 and np.array_equal(got["logits"], again["logits"]) and err < 8e-3
