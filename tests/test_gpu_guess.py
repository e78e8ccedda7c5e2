"""The speculated shift is the last call's, or that of the maximum's running
level where that has been right more often.  Results are the oracle's whatever
the guess; on constant inputs the guess settles, from above and from below, from
one octave away and from many, also where the maximum is a power of two or one
below it; and the level is chosen where single calls leave its octave, the last
call where the maximum drifts."""
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


def expected(maxima, target=7):
    """(level, trust, bp, hint, misses) after each call, from the rule's own
    terms: the level is the bitwidth and the fraction below its leading bit, in
    256ths (maxima below 2^24, which float32 holds exactly)."""
    level = trust = bp = hint = misses = 0
    rows = []
    for mx in maxima:
        b = int(mx).bit_length()
        now = max(b - target, 0)
        misses += hint != now
        lv = (max(b, 1) << 8) + ((max(mx, 1) << 8 >> max(b - 1, 0)) & 255)
        was = max((level >> 8) - target, 0)
        trust = min(max(trust + (was == now) - (bp == now), -3), 3)
        d = lv - level
        level = lv if abs(d) >= 384 else level + ((d + 3 * (d > 0)) >> 2)
        bp = now
        hint = max((level >> 8) - target, 0) if trust > 0 else bp
        rows.append((level, trust, bp, hint, misses))
    return rows


@pytest.mark.parametrize("maxima,chosen", [([8300, 8100, 8400] * 6, True), ([8150, 8200, 7900, 8000] * 5, True),
                                           ([100 << (i // 2) for i in range(14)], False),
                                           ([5000, 0, 5000, 1, 0, 70000, 2, 3], False)])
def test_guess_follows_the_better_of_level_and_last_call(maxima, chosen):
    import torch
    say("guess", maxima[:4])
    K = 8192
    Bd = dev(np.ones((8, K), np.int8))
    C = torch.empty((4, 8), dtype=torch.int8, device="cuda")
    stats = niti.new_stats()
    rows = expected(maxima)
    assert any(hint != bp for _, _, bp, hint, _ in rows) == chosen
    for call, mx in enumerate(maxima):
        A = np.zeros((4, K), np.int8)
        A[2, :mx // 127] = 127
        A[2, mx // 127] = mx % 127
        niti.gemm_fwd(dev(A), Bd, C, stats)
        got = niti.read_stats(stats)[0]
        assert got["max_abs"] == mx
        assert tuple(got[f] for f in ("level", "trust", "bp", "bp_hint", "misses")) == rows[call], (call, got)
