"""The general implicit-GEMM kernel, the small-product kernel and the ring
kernel's stores on rows that are only byte aligned: pieces that cross a row's
end, a filter row's end, the image border and the tensor's first and last
bytes; tile counts on both sides of the 64 x 64 rule; every rounding mode
(stochastic rounding runs all its products there).  Exact against the
oracle."""
import pytest

import oracle
from paper_2009_13108_amd import inputs as I
from paper_2009_13108_amd import niti
from helpers import dev, host, krsc, nchw, nhwc, same_stats, say

pytestmark = pytest.mark.gpu

GEMMS = [
    # M, N, K, relu, mode
    (1, 1, 15, False, oracle.PSR), (3, 2, 17, True, oracle.PSR), (5, 33, 31, False, oracle.RTN),
    (40, 70, 1111, True, oracle.PSR), (1025, 1029, 1, False, oracle.PSR), (1030, 64, 63, True, oracle.SR),
    (1100, 1500, 1111, True, oracle.PSR), (1920, 2176, 65, False, oracle.PSR), (2049, 2040, 257, True, oracle.RTN),
    # small products in 64 rows: one batch of loads, then two and three (2048 bytes each), the last one ragged
    (33, 8064, 48, True, oracle.PSR), (100, 4104, 33, False, oracle.PSR), (130, 2600, 1090, True, oracle.RTN),
    (1000, 520, 64, False, oracle.PSR), (64, 8060, 129, True, oracle.PSR),
    (128, 4096, 4112, True, oracle.PSR), (130, 2600, 2200, False, oracle.RTN), (65, 4101, 2047, True, oracle.PSR),
    (33, 4130, 2049, False, oracle.PSR),
    (1111, 70, 321, False, oracle.SR), (2048, 2176, 127, False, oracle.SR),
]


@pytest.mark.parametrize("case", GEMMS)
def test_products_of_unaligned_rows(case):
    import torch
    M, N, K, relu, mode = case
    say("unaligned gemm", case)
    A, B = I.weights(71, (M, K)), I.weights(72, (N, K))
    C = torch.empty((M, N), dtype=torch.int8, device="cuda")
    stats = niti.new_stats()
    niti.set_sr_seed(stats, 3)
    Ad, Bd = dev(A), dev(B)
    for call in range(2):
        exp, _, st = oracle.gemm_fwd(A, B, relu=relu, mode=mode, sr_seed=3, sr_call=call)
        C.fill_(77)
        niti.gemm_fwd(Ad, Bd, C, stats, relu=relu, mode=mode)
        assert (host(C) == exp).all() and same_stats(niti.read_stats(stats)[0], st), call


CONVS = [
    # n, c, h, w, k, r, s, stride, pad, mode
    (1, 4, 3, 3, 1, 3, 3, 1, 1, oracle.SR), (2, 20, 5, 7, 9, 3, 3, 1, 1, oracle.PSR),
    (3, 36, 9, 8, 33, 5, 5, 2, 2, oracle.PSR), (2, 20, 7, 6, 130, 7, 7, 1, 3, oracle.RTN),
    (2, 68, 6, 6, 66, 1, 1, 2, 0, oracle.PSR), (2, 64, 8, 9, 64, 3, 3, 1, 1, oracle.SR),
    (1, 100, 5, 5, 10, 5, 3, 1, 2, oracle.SR), (9, 20, 60, 60, 200, 3, 3, 1, 1, oracle.PSR),
]


@pytest.mark.parametrize("case", CONVS)
def test_convolutions_of_unaligned_rows(case):
    import torch
    n, c, h, w, k, r, s, stride, pad, mode = case
    say("unaligned conv", case)
    d = oracle.conv_desc(n, c, h, w, k, r, s, stride, pad)
    gd = niti.ConvDesc.make(n, h, w, c, k, r, s, stride, pad)
    P, Q = oracle.conv_out_hw(d)
    x, wt, dy = I.weights(73, (n, c, h, w)), I.weights(74, (k, c, r, s)), I.errors8(75, (n, k, P, Q))
    y = torch.empty(gd.y_shape(), dtype=torch.int8, device="cuda")
    dx = torch.empty(gd.x_shape(), dtype=torch.int8, device="cuda")
    stats = niti.new_stats(2)
    niti.set_sr_seed(stats, 4)
    ws = niti.new_workspace(max(niti.workspace_bytes(op, gd) for op in (niti.OP_CONV_FWD, niti.OP_CONV_BWD_DATA)))
    xd, wd, dyd = dev(nhwc(x)), dev(krsc(wt)), dev(nhwc(dy))
    for call in range(2):
        y_exp, _, st_f = oracle.conv_fwd(d, x, wt, relu=True, mode=mode, sr_seed=4, sr_call=call)
        dx_exp, _, st_b = oracle.conv_bwd_data(d, dy, wt, mode=mode, relu_src=x, sr_seed=4, sr_call=call)
        y.fill_(77)
        dx.fill_(77)
        niti.conv_fwd(gd, xd, wd, y, stats, relu=True, mode=mode, stats_index=0, ws=ws)
        niti.conv_bwd_data(gd, dyd, wd, dx, stats, ws, relu_src=xd, mode=mode, stats_index=1)
        got = niti.read_stats(stats)
        assert (nchw(host(y)) == y_exp).all() and same_stats(got[0], st_f), call
        assert (nchw(host(dx)) == dx_exp).all() and same_stats(got[1], st_b), call


# The ring kernel's output rows at odd addresses: whole pieces and tails of 1
# to 15 bytes, in every tile shape.  The bytes around the output stay as they
# were.
RING = [
    # M, N, K, relu, mode
    (1025, 1111, 16, True, oracle.PSR), (1026, 1030, 64, False, oracle.RTN), (9001, 33, 48, True, oracle.PSR),
    (9000, 63, 272, False, oracle.PSR), (17000, 17, 144, False, oracle.PSR), (17001, 101, 128, True, oracle.PSR),
    (4097, 1039, 272, True, oracle.PSR), (13000, 1011, 32, False, oracle.RTN), (16385, 250, 400, False, oracle.PSR),
    (52000, 255, 64, True, oracle.PSR), (6700, 2037, 160, False, oracle.PSR),
]


@pytest.mark.parametrize("case", RING)
def test_ring_products_with_unaligned_outputs(case):
    import torch
    M, N, K, relu, mode = case
    say("unaligned ring output", case)
    A, B = I.activations(76, (M, K)), I.weights(77, (N, K))
    buf = torch.full((M * N + 64,), 77, dtype=torch.int8, device="cuda")
    C = buf[32:32 + M * N].view(M, N)
    stats = niti.new_stats()
    exp, _, st = oracle.gemm_fwd(A, B, relu=relu, mode=mode)
    Ad, Bd = dev(A), dev(B)
    for call in range(2):
        buf.fill_(77)
        niti.gemm_fwd(Ad, Bd, C, stats, relu=relu, mode=mode)
        assert (host(C) == exp).all() and same_stats(niti.read_stats(stats)[0], st), call
        assert bool((buf[:32] == 77).all()) and bool((buf[32 + M * N:] == 77).all())


@pytest.mark.parametrize("case", [
    # n, c, h, w, k, r, s, stride, pad: the mask and the zeros of strided classes at odd addresses
    (2, 36, 9, 8, 64, 3, 3, 1, 1), (2, 68, 10, 9, 128, 3, 3, 2, 1), (3, 132, 7, 9, 64, 1, 1, 2, 0),
    (40, 20, 28, 27, 192, 3, 3, 1, 1), (40, 100, 28, 27, 64, 3, 3, 2, 1),
])
def test_ring_back_propagation_into_unaligned_rows(case):
    import torch
    n, c, h, w, k, r, s, stride, pad = case
    say("unaligned ring conv", case)
    d = oracle.conv_desc(n, c, h, w, k, r, s, stride, pad)
    gd = niti.ConvDesc.make(n, h, w, c, k, r, s, stride, pad)
    P, Q = oracle.conv_out_hw(d)
    x, wt, dy = I.weights(78, (n, c, h, w)), I.weights(79, (k, c, r, s)), I.errors8(80, (n, k, P, Q))
    exp, _, st = oracle.conv_bwd_data(d, dy, wt, relu_src=x)
    size = n * h * w * c
    buf = torch.full((size + 64,), 77, dtype=torch.int8, device="cuda")
    dx = buf[32:32 + size].view(gd.x_shape())
    stats = niti.new_stats()
    ws = niti.new_workspace(niti.workspace_bytes(niti.OP_CONV_BWD_DATA, gd))
    xd, wd, dyd = dev(nhwc(x)), dev(krsc(wt)), dev(nhwc(dy))
    for call in range(2):
        buf.fill_(77)
        niti.conv_bwd_data(gd, dyd, wd, dx, stats, ws, relu_src=xd)
        assert (nchw(host(dx)) == exp).all() and same_stats(niti.read_stats(stats)[0], st), call
        assert bool((buf[:32] == 77).all()) and bool((buf[32 + size:] == 77).all())
