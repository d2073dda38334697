"""Selection at the edges of its passes and of the rule that gives few frames half the threads."""
import numpy as np
import pytest
import torch

import oracle
from paper_2507_14959_amd import binding, synth
from test_gpu_select import gpu_select

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("F", [1, 63, 64, 65, 255, 256, 257, 513, 1025, 2049])
@pytest.mark.parametrize("K,M", [(64, 20), (80, 30), (80, 45), (126, 64)])
@pytest.mark.parametrize("copy", [False, True])
def test_against_the_oracle(F, K, M, copy):
    rng = np.random.default_rng(F + K)
    mem, acc = synth.make_cover_instance(K, K, M, max_size=6, with_acc=True)
    Y, cur = np.zeros((F, K), dtype=bool), np.zeros(K, dtype=bool)
    for t in range(F):                                   # scenes of a few frames and, at times, long ones
        if rng.random() < (0.4 if t % 300 < 200 else 0.01):
            cur = np.zeros(K, dtype=bool)
            cur[rng.choice(K, size=int(rng.integers(0, 9)), replace=False)] = True
        Y[t] = cur
    scores = np.where(Y, 0.9, 0.1).astype(np.float32)
    o_state = oracle.SelectState(K, M)
    g_state = torch.zeros(binding.poly_select_state_bytes(K), dtype=torch.uint8, device="cuda")
    for part in (scores, scores[::-1].copy()):                  # the second call starts from the state of the first
        o_off, o_ids, o_unc = oracle.select(part, mem, acc=acc, tau=0.3, context_copy=copy, state=o_state)
        off, ids, n, unc = gpu_select(part, mem, acc=acc, tau=0.3, context_copy=copy, state=g_state)
        assert np.array_equal(off, o_off) and np.array_equal(ids, o_ids) and n == len(o_ids) and unc == o_unc
