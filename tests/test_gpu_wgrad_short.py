"""Weight gradients with short reductions, which form g32 twice instead of
storing it: byte-gathered 32 x 32 tiles (few weights) and the LDS-staged
kernel run for the maximum and again for the update (many weights).  Exact
against the oracle at tile remainders, at the limits of both rules and one
past them, in every rounding mode, with and without g32_out and without a
workspace of the caller's."""
import pytest

import oracle
from paper_2009_13108_amd import inputs as I
from paper_2009_13108_amd import niti
from helpers import dev, host, kcrs, krsc, nhwc, same_stats, say

pytestmark = pytest.mark.gpu

CASES = [
    # n, h, w, c, k, mode, mu
    (1, 1, 1, 4, 1, oracle.PSR, 5),
    (31, 1, 1, 20, 33, oracle.RTN, 5),
    (33, 1, 1, 36, 31, oracle.SR, 4),
    (256, 1, 1, 84, 10, oracle.PSR, 3),
    (3, 5, 7, 12, 40, oracle.PSR, 5),            # a 1 x 1 convolution
    (1024, 1, 1, 32, 64, oracle.PSR, 8),         # the most samples of the gathered form
    (1025, 1, 1, 32, 64, oracle.PSR, 1),         # one more
    (8, 1, 1, 512, 512, oracle.SR, 5),           # the most tiles of the gathered form in whole 16s
    (8, 1, 1, 528, 512, oracle.PSR, 5),          # one column of tiles more: through LDS
    (9, 1, 1, 2720, 166, oracle.RTN, 5),         # the other channel counts: 510 tiles, below 128 samples
    (9, 1, 1, 2752, 166, oracle.SR, 5),          # 516: the general kernel
    (128, 1, 1, 5460, 166, oracle.PSR, 5),       # 1026, 128 samples: the general kernel
    (128, 1, 1, 5428, 166, oracle.PSR, 5),       # 1020: gathered
    (8, 1, 1, 1024, 1024, oracle.SR, 5),
    (8, 1, 1, 1040, 1024, oracle.PSR, 5),
    (70, 1, 1, 2064, 528, oracle.RTN, 4),        # ragged tiles and stages
    (65, 1, 1, 1056, 1008, oracle.SR, 5),
    (512, 1, 1, 1296, 816, oracle.PSR, 5),       # the most samples of that form
    (513, 1, 1, 1296, 816, oracle.PSR, 5),       # one more
    (16, 1, 1, 8208, 144, oracle.PSR, 5),
    (40, 1, 1, 16400, 64, oracle.RTN, 5),        # 64-channel tiles
]


@pytest.mark.parametrize("case", CASES)
def test_short_reductions(case):
    import torch
    n, h, w, c, k, mode, mu = case
    say("short wgrad", case)
    d = oracle.conv_desc(n, c, h, w, k, 1, 1, 1, 0)
    gd = niti.ConvDesc.make(n, h, w, c, k, 1, 1, 1, 0)
    x, wt = I.activations(41, (n, c, h, w)), I.weights(42, (k, c, 1, 1))
    dy = I.errors8(43, (n, k, h, w))
    ws = niti.new_workspace(niti.workspace_bytes(niti.OP_CONV_BWD_WEIGHT, gd))
    xd, dyd = dev(nhwc(x)), dev(nhwc(dy))
    stats = niti.new_stats(3)
    niti.set_sr_seed(stats, 5)
    g32 = torch.empty(gd.w_shape(), dtype=torch.int32, device="cuda")
    for i, kw in enumerate([{}, {"g32_out": g32}, {"noalloc": True}]):
        wd, prev = dev(krsc(wt)), wt
        noalloc = kw.pop("noalloc", False)
        if noalloc and niti.workspace_bytes(niti.OP_CONV_BWD_WEIGHT, gd) > niti.NOALLOC_SCRATCH_BYTES:
            continue
        for call in range(2):   # the second call runs on the first one's statistics
            exp_w, exp_g, st = oracle.conv_bwd_weight(d, x, dy, prev, mu=mu, mode=mode, sr_seed=5, sr_call=call)
            if noalloc:
                niti.conv_bwd_weight_noalloc(gd, xd, dyd, wd, stats, mu=mu, mode=mode, stats_index=i)
            else:
                niti.conv_bwd_weight(gd, xd, dyd, wd, stats, ws, mu=mu, mode=mode, stats_index=i, **kw)
            assert (kcrs(host(wd)) == exp_w).all(), (i, call)
            assert same_stats(niti.read_stats(stats)[i], st), (i, call)
            if "g32_out" in kw:
                assert (kcrs(host(g32)) == exp_g).all()
            prev = exp_w


@pytest.mark.parametrize("case", [
    # n, c, h, w, k, r, s, stride, pad, mode: convolutions formed twice
    (1, 96, 4, 4, 112, 3, 3, 1, 1, oracle.PSR),
    (1, 160, 3, 3, 112, 3, 3, 1, 1, oracle.SR),
    (2, 96, 9, 8, 144, 3, 3, 2, 1, oracle.RTN),
    (1, 80, 6, 5, 48, 5, 5, 1, 2, oracle.PSR),
    (3, 208, 9, 9, 400, 1, 1, 2, 0, oracle.PSR),
])
def test_convolutions_formed_twice(case):
    n, c, h, w, k, r, s, stride, pad, mode = case
    say("short conv wgrad", case)
    d = oracle.conv_desc(n, c, h, w, k, r, s, stride, pad)
    gd = niti.ConvDesc.make(n, h, w, c, k, r, s, stride, pad)
    P, Q = oracle.conv_out_hw(d)
    x, wt, dy = I.activations(44, (n, c, h, w)), I.weights(45, (k, c, r, s)), I.errors8(46, (n, k, P, Q))
    exp_w, _, st = oracle.conv_bwd_weight(d, x, dy, wt, mu=5, mode=mode, sr_seed=6, sr_call=0)
    stats = niti.new_stats()
    niti.set_sr_seed(stats, 6)
    wd = dev(krsc(wt))
    niti.timing_enable(True)
    niti.conv_bwd_weight(gd, dev(nhwc(x)), dev(nhwc(dy)), wd, stats,
                         niti.new_workspace(niti.workspace_bytes(niti.OP_CONV_BWD_WEIGHT, gd)), mu=5, mode=mode)
    niti.timing_enable(False)
    assert (kcrs(host(wd)) == exp_w).all() and same_stats(niti.read_stats(stats)[0], st)
    assert not [1 for fam, _, _ in niti.timing_records() if fam == niti.TIMING_SUM]   # g32 was not stored
