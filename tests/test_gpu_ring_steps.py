"""The ring kernel's K steps and tiles at their edges, exact against the
oracle: reductions that end inside a 64- and a 128-byte step, one step, one
more than the ring holds; channels in whole 128s, whole 64s and both in one
layer's two directions; tile counts on both sides of one tile per CU; output
channels that 256-column tiles pad further than 128-column ones, in either."""
import pytest

import oracle
from paper_2009_13108_amd import inputs as I
from paper_2009_13108_amd import niti
from helpers import dev, host, krsc, nchw, nhwc, same_stats, say

pytestmark = pytest.mark.gpu

GEMMS = [
    # M, N, K, relu, mode
    (4224, 1030, 16, True, oracle.PSR), (4224, 1030, 112, False, oracle.PSR), (4096, 1100, 128, True, oracle.RTN),
    (4100, 1030, 144, False, oracle.PSR), (4100, 1030, 272, True, oracle.PSR), (33000, 100, 400, True, oracle.PSR),
    (70000, 40, 208, False, oracle.PSR), (2048, 2048, 528, True, oracle.PSR), (2049, 2048, 528, True, oracle.PSR),
    (7000, 2000, 192, False, oracle.PSR), (5200, 2700, 160, True, oracle.RTN), (42000, 320, 144, True, oracle.PSR),
    # steps of 128 bytes: whole ones, and last ones of 16, 64, 80 and 112; then in tiles of 256
    (4224, 1030, 384, True, oracle.PSR), (4100, 1030, 400, False, oracle.PSR), (4100, 1030, 576, True, oracle.RTN),
    (4100, 1030, 464, False, oracle.PSR), (4100, 1030, 496, True, oracle.PSR), (13200, 1000, 640, False, oracle.PSR),
    (13200, 1000, 720, True, oracle.PSR), (12800, 1100, 144, False, oracle.RTN),
]


@pytest.mark.parametrize("case", GEMMS)
def test_products(case):
    import torch
    M, N, K, relu, mode = case
    say("ring gemm", case)
    A, B = I.activations(81, (M, K)), I.weights(82, (N, K))
    C = torch.empty((M, N), dtype=torch.int8, device="cuda")
    stats = niti.new_stats()
    exp, _, st = oracle.gemm_fwd(A, B, relu=relu, mode=mode)
    Ad, Bd = dev(A), dev(B)
    for call in range(2):
        C.fill_(77)
        niti.gemm_fwd(Ad, Bd, C, stats, relu=relu, mode=mode)
        assert (host(C) == exp).all() and same_stats(niti.read_stats(stats)[0], st), call


CONVS = [
    # n, c, h, w, k, r, s, stride, pad, mode
    (3, 128, 9, 11, 192, 3, 3, 1, 1, oracle.PSR), (2, 384, 7, 7, 128, 1, 1, 1, 0, oracle.PSR),
    (42, 128, 29, 28, 160, 3, 3, 1, 1, oracle.PSR), (42, 192, 29, 28, 256, 1, 1, 1, 0, oracle.RTN),
    (11, 256, 57, 55, 320, 1, 1, 2, 0, oracle.PSR), (40, 256, 30, 29, 64, 3, 3, 2, 1, oracle.PSR),
]


@pytest.mark.parametrize("case", CONVS)
def test_convolutions(case):
    import torch
    n, c, h, w, k, r, s, stride, pad, mode = case
    say("ring conv", case)
    d = oracle.conv_desc(n, c, h, w, k, r, s, stride, pad)
    gd = niti.ConvDesc.make(n, h, w, c, k, r, s, stride, pad)
    P, Q = oracle.conv_out_hw(d)
    x, wt, dy = I.activations(83, (n, c, h, w)), I.weights(84, (k, c, r, s)), I.errors8(85, (n, k, P, Q))
    y_exp, _, st_f = oracle.conv_fwd(d, x, wt, relu=True, mode=mode)
    dx_exp, _, st_b = oracle.conv_bwd_data(d, dy, wt, mode=mode, relu_src=x)
    y = torch.empty(gd.y_shape(), dtype=torch.int8, device="cuda")
    dx = torch.empty(gd.x_shape(), dtype=torch.int8, device="cuda")
    stats = niti.new_stats(2)
    ws = niti.new_workspace(max(niti.workspace_bytes(op, gd) for op in (niti.OP_CONV_FWD, niti.OP_CONV_BWD_DATA)))
    xd, wd, dyd = dev(nhwc(x)), dev(krsc(wt)), dev(nhwc(dy))
    for call in range(2):
        y.fill_(77)
        dx.fill_(77)
        niti.conv_fwd(gd, xd, wd, y, stats, relu=True, mode=mode, stats_index=0, ws=ws)
        niti.conv_bwd_data(gd, dyd, wd, dx, stats, ws, relu_src=xd, mode=mode, stats_index=1)
        got = niti.read_stats(stats)
        assert (nchw(host(y)) == y_exp).all() and same_stats(got[0], st_f), call
        assert (nchw(host(dx)) == dx_exp).all() and same_stats(got[1], st_b), call
