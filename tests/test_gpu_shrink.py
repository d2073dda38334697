"""The shrink whose rows stream through LDS: every split of the contraction, runs of rows, branches over workgroups, passes over the ranks."""
import pytest

import test_gpu_small_products as products

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_xblocks,T,K,N,r,per_block", [
    (9, 197, 1536, 520, 16, 3),      # K over four waves, two chunks each; a third branch on workgroups of its own
    (40, 21, 3072, 520, 3, 2),       # four chunks, runs of one subtile, the second one mostly past the end
    (13, 130, 1152, 520, 8, 1),      # K over two waves, three chunks each, runs two by two
    (110, 197, 192, 64, 16, 2),      # K undivided: four runs, no sums to meet
    (31, 197, 1024, 264, 40, 2),      # items of 128 columns; two passes over the ranks, the second one of a single group
    (300, 112, 384, 64, 12, 1),      # a run of seven subtiles and an idle one
    (600, 113, 128, 64, 16, 1),      # one chunk in all, more workgroups than the chip holds
    (1100, 33, 256, 64, 5, 3),       # more input blocks than the CSR form takes: row maps from a launch before
])
def test_against_the_oracle(n_xblocks, T, K, N, r, per_block):
    products.test_against_the_oracle(n_xblocks, T, K, N, r, per_block)
