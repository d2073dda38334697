"""Products whose 32-row subtiles hold several token blocks: as many as are fetched ahead, and more."""
import pytest

from paper_2507_14959_amd import synth
from test_gpu_forward import compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,D,heads,Dm,hw,r,L0", [
    (synth.DT_F32, 64, 1, 128, 16, 4, 0),       # 5 tokens: seven or eight blocks
    (synth.DT_F32, 128, 2, 256, 24, 20, 1),     # 10 tokens, a second step of ranks
    (synth.DT_F32, 192, 3, 192, 32, 6, 0),      # 17 tokens: two or three; a rank that fills no load
    (synth.DT_F32, 64, 1, 128, 80, 8, 0),       # 101 tokens: one or two
    (synth.DT_BF16, 512, 8, 512, 16, 20, 0),
    (synth.DT_BF16, 512, 8, 1024, 24, 8, 1),
])
@pytest.mark.parametrize("compose", ["branch", "sum"])
def test_against_the_oracle(dtype, D, heads, Dm, hw, r, L0, compose):
    cfg, w, frames, off, ids = synth.make_small_case(11 + D + hw, dtype=dtype, targets=15, L=2, F=7, r=r, max_set=3, n_adapters=5, D=D, heads=heads, Dm=Dm,
                                                     hw=hw, patch=8)
    # bf16: 1.6e-3 to 2.9e-3; a bias left out of one linear of a layer moves the logits by 1.3e-2 and more
    compare(cfg, w, frames, off, ids, L0, compose=compose, tol=8e-3 if dtype == synth.DT_BF16 else None)
