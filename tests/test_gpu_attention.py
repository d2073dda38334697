"""Attention of long blocks with two query tiles per wave: more (block, head) pairs than CUs."""
import pytest

from paper_2507_14959_amd import synth
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
    compare(cfg, w, frames, off, ids, L0)
