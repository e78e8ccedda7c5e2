"""The speculated shift follows the maximum's running level: results are the
oracle's whatever the guess, and on constant inputs the guess settles, from
above and from below, from one octave away and from many, also where the
maximum is a power of two or one below it."""
import numpy as np
import pytest

import oracle
from paper_2009_13108_amd import niti
from helpers import dev, host, same_stats, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tops", [(1 << 14, (1 << 14) - 1, 1 << 14), (1 << 10, 1 << 20, 1 << 9), (3 << 12, 1 << 12, 5 << 12),
                                  (200, 127, 0, 4097), (1 << 12, (1 << 13) - 1, 1 << 12)])
def test_guess_settles_on_constant_inputs(tops):
    import torch
    say("guess", tops)
    K = 4096
    B = np.full((8, K), 1, np.int8)
    stats = niti.new_stats()
    C = torch.empty((4, 8), dtype=torch.int8, device="cuda")
    for top in tops:
        # rows whose sums are exactly the wanted maximum and small values
        A = np.zeros((4, K), np.int8)
        v, left = 0, top
        scale = max(1, -(-top // (K * 127)))
        while left > 0 and v < K:
            A[0, v] = min(127, left // scale if left >= scale else left)
            left -= int(A[0, v]) * scale
            v += 1
        Bs = (B * min(scale, 127)).astype(np.int8)
        A[1, :5] = 1
        exp, _, st = oracle.gemm_fwd(A, Bs)
        Ad, Bd = dev(A), dev(Bs)
        for call in range(14):
            C.fill_(77)
            niti.gemm_fwd(Ad, Bd, C, stats)
            assert (host(C) == exp).all() and same_stats(niti.read_stats(stats)[0], st), (top, call)
            if call == 11:
                settled = niti.read_stats(stats)[0]["misses"]
        assert niti.read_stats(stats)[0]["misses"] == settled, top
