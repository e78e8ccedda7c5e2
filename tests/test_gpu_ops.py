"""GPU parity of every C-ABI entry point against the CPU oracle.

Each case draws seeded inputs, runs the HIP library through its C ABI and
the oracle on the same bytes, and requires byte-identical int8 outputs,
identical int32 gradients and identical block statistics (max, b, bp) and
exponents.  Sizes span several tiles with ragged edges; each case is also
run twice so the second call exercises the speculated-shift path.
"""
import numpy as np
import pytest

import oracle
from paper_2009_13108_amd import inputs as I
from paper_2009_13108_amd import niti
from helpers import dev, host, kcrs, krsc, nchw, nhwc, say, same_stats

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _lib():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    niti.lib()


def _i8(v):
    import torch
    return torch.tensor([v], dtype=torch.int8, device="cuda")


GEMM_CASES = [
    # M, N, K, relu, mode, distribution of B
    (1, 1, 1, False, oracle.PSR, "w"),
    (7, 5, 3, False, oracle.PSR, "w"),
    (33, 17, 65, True, oracle.PSR, "w"),
    (32, 128, 784, False, oracle.PSR, "e5"),
    (300, 200, 784, True, oracle.PSR, "w"),
    (257, 129, 1000, False, oracle.RTN, "w"),
    (64, 10, 128, False, oracle.PSR, "w"),
    (129, 300, 0, False, oracle.PSR, "w"),
    (513, 257, 333, True, oracle.PSR, "e5"),
    (3000, 64, 128, False, oracle.PSR, "w"),      # 256x64 tiles
    (70001, 100, 64, True, oracle.PSR, "w"),      # 128x128 tiles, ragged M and N
    (4100, 4096, 272, False, oracle.PSR, "w"),    # 256x256 tiles, ragged M and K
    (2000, 300, 512, False, oracle.RTN, "e5"),    # 128x128 tiles
    # few outputs, long reduction: reduction split over the waves of a tile
    (128, 1000, 512, False, oracle.PSR, "w"),     # classifier head forward
    (128, 512, 1000, True, oracle.PSR, "e5"),     # rows of 1000 bytes (8-byte aligned)
    (96, 40, 5000, False, oracle.RTN, "w"),       # several load batches per wave
    (1024, 66, 77, True, oracle.PSR, "w"),        # largest row count of that path
    (1025, 30, 200, False, oracle.PSR, "w"),      # one row more: tiled kernels
]


@pytest.mark.parametrize("case", GEMM_CASES)
def test_gemm_fwd_parity(case):
    import torch
    M, N, K, relu, mode, dist = case
    say("gemm_fwd", case)
    A = I.activations(1000 + M, (M, K))
    B = (I.weights if dist == "w" else I.errors5)(2000 + N, (N, K))
    exp_out, _, st = oracle.gemm_fwd(A, B, relu=relu, mode=mode)
    s_exp, _ = oracle.out_exponent(-7, -9, st["bp"])
    dA, dB = dev(A), dev(B)
    C = torch.empty((M, N), dtype=torch.int8, device="cuda")
    stats = niti.new_stats()
    sa, sb, sc = _i8(-7), _i8(-9), _i8(0)
    for rep in range(2):
        C.fill_(99)
        niti.gemm_fwd(dA, dB, C, stats, sa, sb, sc, 7, relu, mode)
        torch.cuda.synchronize()
        g = niti.read_stats(stats)[0]
        assert (host(C) == exp_out).all(), "rep %d" % rep
        assert same_stats(g, st), (g, st)
        assert int(host(sc)[0]) == s_exp
        assert g["calls"] == rep + 1
    assert g["misses"] <= 1 and g["flags"] & niti.FLAG_HINT_MISS == 0


def test_gemm_fwd_hint_miss_recomputes():
    import torch
    say("gemm_fwd hint miss")
    # One stats block reused across tensors with different block exponents:
    # every call's first guess is wrong and the output must be recomputed.
    A1 = I.activations(1, (64, 256)); B1 = I.weights(2, (96, 256))
    A2 = I.errors5(3, (64, 256)); B2 = I.errors5(4, (96, 256))
    stats = niti.new_stats()
    for (A, B) in [(A1, B1), (A2, B2), (A1, B1)]:
        exp_out, _, st = oracle.gemm_fwd(A, B)
        C = torch.empty((64, 96), dtype=torch.int8, device="cuda")
        niti.gemm_fwd(dev(A), dev(B), C, stats)
        torch.cuda.synchronize()
        g = niti.read_stats(stats)[0]
        assert (host(C) == exp_out).all() and same_stats(g, st)
        assert g["flags"] & niti.FLAG_HINT_MISS


CONV_CASES = [
    # n, c, h, w, k, r, s, stride, pad, relu
    (1, 4, 5, 5, 4, 3, 3, 1, 1, False),
    (2, 4, 7, 6, 8, 3, 3, 1, 1, True),
    (2, 8, 9, 9, 12, 3, 3, 2, 1, False),
    (1, 4, 11, 11, 8, 7, 7, 2, 3, True),
    (2, 4, 8, 8, 20, 1, 1, 2, 0, False),
    (1, 8, 6, 7, 12, 1, 1, 1, 0, True),
    (3, 4, 5, 5, 4, 3, 3, 1, 0, False),
    (1, 4, 6, 6, 8, 2, 3, 2, 2, False),
    (2, 64, 14, 14, 64, 3, 3, 1, 1, True),
    (2, 64, 15, 15, 128, 3, 3, 2, 1, False),
    (2, 32, 16, 16, 96, 1, 1, 2, 0, True),
    (1, 4, 32, 32, 64, 7, 7, 2, 3, True),
    (4, 128, 7, 7, 130, 3, 3, 1, 1, False),
    # 64 input channels, stride 1: weights in registers, rows staged per block
    (3, 64, 9, 7, 48, 3, 3, 1, 1, False),
    (1, 64, 5, 5, 64, 3, 3, 1, 0, True),
    (5, 64, 13, 11, 64, 3, 3, 1, 1, True),
    # few channels: padded-copy window path (s*c <= 64), windows of 16/32/64 bytes
    (2, 12, 9, 9, 16, 3, 3, 1, 1, True),
    (2, 8, 10, 10, 32, 3, 3, 2, 1, False),
    (3, 4, 13, 12, 48, 5, 5, 2, 2, True),
    (2, 16, 7, 7, 32, 2, 2, 1, 0, False),
    # no padding and rows that reach the last window: read in place (an image
    # stored with its zero border); one column short: copied
    (2, 4, 38, 38, 64, 7, 7, 2, 0, True),
    (2, 4, 37, 37, 64, 7, 7, 2, 0, False),
    # strided 3x3 back-propagation over 64 error channels (odd sizes: sub-pixel
    # classes of unequal size)
    (2, 32, 9, 11, 64, 3, 3, 2, 1, True),
    (1, 64, 8, 8, 128, 3, 3, 2, 1, False),
    (2, 128, 13, 13, 256, 3, 3, 2, 1, True),
    # strided 1x1: three of four sub-pixel classes have no taps
    (2, 64, 14, 14, 128, 1, 1, 2, 0, True),
    (2, 64, 7, 9, 256, 1, 1, 2, 0, False),
    (2, 256, 9, 7, 128, 1, 1, 2, 0, True),
    # 1x1 over padding only: no class has taps, dx is all zeros
    (1, 4, 1, 1, 8, 1, 1, 2, 1, False),
    # classifier head as a 1x1 convolution: 512 features, 1000 classes
    (128, 512, 1, 1, 1000, 1, 1, 1, 0, True),
    # stride 1, 64 or 128 channels: input rows staged per band of output rows
    # (ragged last band, two or three 64-channel output tiles)
    (2, 64, 20, 60, 64, 3, 3, 1, 1, True),
    (2, 128, 30, 20, 128, 3, 3, 1, 1, False),
    (1, 64, 9, 7, 192, 3, 3, 1, 1, True),
    (3, 128, 6, 9, 64, 3, 3, 1, 0, False),
    (1, 64, 11, 13, 64, 5, 5, 1, 2, True),
]


def _conv_inputs(case, seed):
    n, c, h, w, k, r, s, st, pd, relu = case
    d = oracle.conv_desc(n, c, h, w, k, r, s, st, pd)
    P, Q = oracle.conv_out_hw(d)
    x = I.activations(seed + 1, (n, c, h, w))
    wt = I.weights(seed + 2, (k, c, r, s))
    dy = I.errors8(seed + 3, (n, k, P, Q))
    gd = niti.ConvDesc.make(n, h, w, c, k, r, s, st, pd)
    return d, gd, x, wt, dy


@pytest.mark.parametrize("case", CONV_CASES)
def test_conv_fwd_parity(case):
    import torch
    say("conv_fwd", case)
    d, gd, x, wt, dy = _conv_inputs(case, 10 * case[1] + case[4])
    relu = case[-1]
    exp_out, _, st = oracle.conv_fwd(d, x, wt, relu=relu)
    s_exp, _ = oracle.out_exponent(-3, -8, st["bp"])
    y = torch.empty(gd.y_shape(), dtype=torch.int8, device="cuda")
    stats = niti.new_stats()
    sx, sw, sy = _i8(-3), _i8(-8), _i8(0)
    dx_, dw_ = dev(nhwc(x)), dev(krsc(wt))
    nws = niti.workspace_bytes(niti.OP_CONV_FWD, gd)
    ws = niti.new_workspace(nws) if nws else None
    for rep in range(2):
        y.fill_(77)
        niti.conv_fwd(gd, dx_, dw_, y, stats, sx, sw, sy, relu=relu, ws=ws)
        torch.cuda.synchronize()
        g = niti.read_stats(stats)[0]
        assert (nchw(host(y)) == exp_out).all(), "rep %d" % rep
        assert same_stats(g, st) and int(host(sy)[0]) == s_exp


@pytest.mark.parametrize("case", CONV_CASES)
def test_conv_bwd_data_parity(case):
    import torch
    say("conv_bwd_data", case)
    d, gd, x, wt, dy = _conv_inputs(case, 7 * case[2] + case[4])
    use_mask = case[-1]
    relu_src = I.weights(55, (d.n, d.c, d.h, d.w)) if use_mask else None
    exp_out, _, st = oracle.conv_bwd_data(d, dy, wt, relu_src=relu_src)
    dx = torch.empty(gd.x_shape(), dtype=torch.int8, device="cuda")
    stats = niti.new_stats()
    ws = niti.new_workspace(niti.workspace_bytes(niti.OP_CONV_BWD_DATA, gd))
    mask = dev(nhwc(relu_src)) if use_mask else None
    for rep in range(2):
        dx.fill_(55)
        niti.conv_bwd_data(gd, dev(nhwc(dy)), dev(krsc(wt)), dx, stats, ws, relu_src=mask)
        torch.cuda.synchronize()
        g = niti.read_stats(stats)[0]
        assert (nchw(host(dx)) == exp_out).all(), "rep %d" % rep
        assert same_stats(g, st)


@pytest.mark.parametrize("case", CONV_CASES)
def test_conv_bwd_data_packed_parity(case):
    """The filter packed once, then changed in place: the packed calls still
    compute the back-propagation of the filter as it was packed."""
    import torch
    say("conv_bwd_data_packed", case)
    d, gd, x, wt, dy = _conv_inputs(case, 5 * case[2] + case[4])
    use_mask = case[-1]
    relu_src = I.weights(57, (d.n, d.c, d.h, d.w)) if use_mask else None
    exp_out, _, st = oracle.conv_bwd_data(d, dy, wt, relu_src=relu_src)
    dx = torch.empty(gd.x_shape(), dtype=torch.int8, device="cuda")
    stats = niti.new_stats()
    packed = niti.new_workspace(niti.workspace_bytes(niti.OP_CONV_BWD_DATA, gd))
    packed.fill_(0x5A)
    w = dev(krsc(wt))
    mask = dev(nhwc(relu_src)) if use_mask else None
    niti.conv_pack_bwd_data(gd, w, packed)
    w.fill_(3)
    for rep in range(2):
        dx.fill_(55)
        niti.conv_bwd_data_packed(gd, dev(nhwc(dy)), packed, dx, stats, relu_src=mask)
        torch.cuda.synchronize()
        g = niti.read_stats(stats)[0]
        assert (nchw(host(dx)) == exp_out).all(), "rep %d" % rep
        assert same_stats(g, st)


@pytest.mark.parametrize("case", CONV_CASES)
@pytest.mark.parametrize("mu", [5, 3])
def test_conv_bwd_weight_parity(case, mu):
    import torch
    say("conv_bwd_weight", case, mu)
    d, gd, x, wt, dy = _conv_inputs(case, 3 * case[3] + case[1])
    exp_w, exp_g32, st = oracle.conv_bwd_weight(d, x, dy, wt, mu=mu)
    w_dev = dev(krsc(wt))
    g32 = torch.empty(gd.w_shape(), dtype=torch.int32, device="cuda")
    stats = niti.new_stats()
    ws = niti.new_workspace(niti.workspace_bytes(niti.OP_CONV_BWD_WEIGHT, gd))
    niti.conv_bwd_weight(gd, dev(nhwc(x)), dev(nhwc(dy)), w_dev, stats, ws, g32_out=g32, mu=mu)
    torch.cuda.synchronize()
    g = niti.read_stats(stats)[0]
    assert (kcrs(host(g32)) == exp_g32).all()
    assert (kcrs(host(w_dev)) == exp_w).all()
    assert same_stats(g, st)
    # same again through the workspace (no g32_out), from the original weights
    w2 = dev(krsc(wt))
    niti.conv_bwd_weight(gd, dev(nhwc(x)), dev(nhwc(dy)), w2, stats, ws, mu=mu)
    torch.cuda.synchronize()
    assert (kcrs(host(w2)) == exp_w).all()


STRIDE_CASES = [
    # n, c, h, w, k, r, s, stride, pad, relu: strides above 2 (forward and
    # weight gradient only), few channels (window copy) and 64 channels
    (2, 4, 31, 29, 32, 11, 11, 4, 2, True),
    (2, 8, 17, 17, 16, 5, 5, 3, 1, False),
    (2, 64, 15, 13, 64, 3, 3, 3, 1, True),
    (1, 128, 16, 16, 96, 3, 3, 4, 0, False),
    (3, 64, 9, 9, 40, 1, 1, 8, 0, True),
]


def test_conv_bordered_image_read_in_place():
    """A few-channel image stored with its zero border (no padding in the
    descriptor, rows reaching the last filter window) is read in place; the
    forward pass and the weight gradient then equal those of the unbordered
    image with the padding in the descriptor, byte for byte, statistics
    included (the 7x7 stride-2 image layer: 32x32 inside a 3-pixel border)."""
    import torch
    n, c, hw, k, r, st, pd = 2, 4, 32, 64, 7, 2, 3
    x = I.activations(901, (n, hw, hw, c))
    x[..., 3:] = 0
    xb = np.zeros((n, hw + 2 * pd, hw + 2 * pd, c), np.int8)
    xb[:, pd:pd + hw, pd:pd + hw] = x
    wt = I.weights(902, (k, r, r, c))
    wt[..., 3:] = 0
    gp = niti.ConvDesc.make(n, hw, hw, c, k, r, r, st, pd)
    gb = niti.ConvDesc.make(n, hw + 2 * pd, hw + 2 * pd, c, k, r, r, st, 0)
    assert gp.y_shape() == gb.y_shape()
    assert niti.workspace_bytes(niti.OP_CONV_FWD, gb) < niti.workspace_bytes(niti.OP_CONV_FWD, gp)
    assert niti.workspace_bytes(niti.OP_CONV_BWD_WEIGHT, gb) < niti.workspace_bytes(niti.OP_CONV_BWD_WEIGHT, gp)
    dy = dev(I.errors8(903, gp.y_shape()))
    res = []
    for gd, xi in ((gp, x), (gb, xb)):
        stats = niti.new_stats(2)
        ws = niti.new_workspace(max(niti.workspace_bytes(op, gd) for op in (niti.OP_CONV_FWD, niti.OP_CONV_BWD_WEIGHT)))
        xd, wd = dev(xi), dev(wt)
        y = torch.empty(gd.y_shape(), dtype=torch.int8, device="cuda")
        g32 = torch.empty(gd.w_shape(), dtype=torch.int32, device="cuda")
        niti.conv_fwd(gd, xd, wd, y, stats, relu=True, ws=ws, stats_index=0)
        niti.conv_bwd_weight(gd, xd, dy, wd, stats, ws, g32_out=g32, mu=5, stats_index=1)
        torch.cuda.synchronize()
        res.append((host(y), host(g32), host(wd), niti.read_stats(stats)))
    (y0, g0, w0, s0), (y1, g1, w1, s1) = res
    assert (y0 == y1).all() and (g0 == g1).all() and (w0 == w1).all()
    for i in (0, 1):
        assert all(int(s0[i][f]) == int(s1[i][f]) for f in ("max_abs", "b", "bp", "flags")), i
    assert y0.any() and g0.any()


@pytest.mark.parametrize("case", STRIDE_CASES)
def test_conv_large_stride_parity(case):
    import torch
    say("conv large stride", case)
    d, gd, x, wt, dy = _conv_inputs(case, 11 * case[2] + case[7])
    relu = case[-1]
    y_o, _, st_f = oracle.conv_fwd(d, x, wt, relu=relu)
    w_o, g_o, st_w = oracle.conv_bwd_weight(d, x, dy, wt, mu=5)
    y = torch.empty(gd.y_shape(), dtype=torch.int8, device="cuda")
    stats = niti.new_stats(2)
    ws = niti.new_workspace(max(16, niti.workspace_bytes(niti.OP_CONV_FWD, gd),
                                niti.workspace_bytes(niti.OP_CONV_BWD_WEIGHT, gd)))
    assert niti.workspace_bytes(niti.OP_CONV_BWD_DATA, gd) == 0
    niti.conv_fwd(gd, dev(nhwc(x)), dev(krsc(wt)), y, stats, relu=relu, ws=ws, stats_index=0)
    w_dev = dev(krsc(wt))
    g32 = torch.empty(gd.w_shape(), dtype=torch.int32, device="cuda")
    niti.conv_bwd_weight(gd, dev(nhwc(x)), dev(nhwc(dy)), w_dev, stats, ws, g32_out=g32, mu=5, stats_index=1)
    torch.cuda.synchronize()
    g = niti.read_stats(stats)
    assert (nchw(host(y)) == y_o).all() and same_stats(g[0], st_f)
    assert (kcrs(host(g32)) == g_o).all()
    assert (kcrs(host(w_dev)) == w_o).all() and same_stats(g[1], st_w)


@pytest.mark.parametrize("n", [0, 1, 5, 1000, 65537])
def test_round_psr_parity(n):
    import torch
    say("round_psr", n)
    x = I.uniform_int(90 + n, (n,), -(1 << 30), (1 << 30), dtype=np.int32)
    if n > 3:
        x[3] = -(2 ** 31)
    exp, st = oracle.shift_round(x, 7)
    y = torch.empty(n, dtype=torch.int8, device="cuda")
    stats = niti.new_stats()
    s_in, s_out = _i8(-5), _i8(0)
    niti.round_psr(dev(x), y, -1, 7, stats, s_in, s_out)
    torch.cuda.synchronize()
    g = niti.read_stats(stats)[0]
    assert (host(y) == exp).all() and same_stats(g, st)
    assert int(host(s_out)[0]) == max(-128, min(127, -5 + st["bp"]))
    for bp in (0, 1, 4, 9, 31):
        niti.round_psr(dev(x), y, bp, 7, None, s_in, s_out)
        torch.cuda.synchronize()
        assert (host(y) == oracle.round_fixed(x, bp)).all()
        assert int(host(s_out)[0]) == -5 + bp
        niti.round_psr(dev(x), y, bp, 7, None, mode=niti.RTN)
        torch.cuda.synchronize()
        assert (host(y) == oracle.round_fixed(x, bp, oracle.RTN)).all()


def test_round_psr_every_shift():
    """Every binary point 0..31, both parities of the fraction split, on the
    full int32 range and on values at the rounding decision (upper half of
    the fraction equal to the lower half, one above, one below)."""
    import torch
    say("round_psr every shift")
    rng = np.random.default_rng(77)
    for bp in range(32):
        odd, h = bp & 1, (bp - (bp & 1)) // 2
        vals = [0, 1, -1, 2 ** 31 - 1, -(2 ** 31), 2 ** 31 - 2, -(2 ** 31) + 1]
        q = rng.integers(0, 128, 64)
        for lo in rng.integers(0, 1 << h, 8) if h else [0]:
            for d in (-1, 0, 1):
                hi_ = min(max(int(lo) + d, 0), (1 << h) - 1) if h else 0
                f = ((hi_ << h) | int(lo)) << odd
                for qq in q[:8]:
                    v = (int(qq) << bp) + f
                    if v < 2 ** 31:
                        vals += [v, -v]
        vals += list(rng.integers(-(2 ** 31), 2 ** 31, 2000))
        x = np.array(vals, dtype=np.int64).astype(np.int32)
        y = torch.empty(x.size, dtype=torch.int8, device="cuda")
        niti.round_psr(dev(x), y, bp, 7, None)
        torch.cuda.synchronize()
        assert (host(y) == oracle.round_fixed(x, bp)).all(), bp


def test_round_psr_worked_examples():
    import json, os, torch
    g = json.load(open(os.path.join(os.path.dirname(__file__), "golden", "psr_examples.json")))
    for c in g["cases"]:
        x = dev(np.array([c["x"]], np.int32))
        y = torch.empty(1, dtype=torch.int8, device="cuda")
        niti.round_psr(x, y, c["bp"], 7)
        torch.cuda.synchronize()
        assert int(host(y)[0]) == c["out"], c
    for c in g["blocks"]:
        x = dev(np.array(c["acc"], np.int32))
        y = torch.empty(len(c["acc"]), dtype=torch.int8, device="cuda")
        stats = niti.new_stats()
        niti.round_psr(x, y, -1, c["target"], stats)
        torch.cuda.synchronize()
        assert host(y).tolist() == c["out"] and niti.read_stats(stats)[0]["bp"] == c["bp"]


@pytest.mark.parametrize("s_a", [-128, -55, -54, -40, -31, -23, -22, -13, -9, -7, -6, -3, 0, 5, 15, 16, 100])
@pytest.mark.parametrize("shape", [(256, 10), (128, 1000), (3, 65), (5, 1024), (4, 1500)])
def test_int_ce_loss_grad_parity(s_a, shape):
    import torch
    say("loss", s_a, shape)
    B, N = shape
    logits = I.weights(500 + B + s_a, (B, N))
    labels = I.labels(600 + N, B, N)
    err = torch.empty((B, N), dtype=torch.int8, device="cuda")
    stats = niti.new_stats()
    ws = niti.new_workspace(niti.workspace_bytes(niti.OP_INT_CE_LOSS, None, B, N))
    for mode in (niti.PSR, niti.RTN):
        exp, _, st = oracle.int_ce_loss_grad(logits, s_a, labels, mode=mode)
        err.fill_(99)
        niti.int_ce_loss_grad(dev(logits), _i8(s_a), dev(labels), err, stats, ws, mode=mode)
        torch.cuda.synchronize()
        g = niti.read_stats(stats)[0]
        assert (host(err) == exp).all(), mode
        assert same_stats(g, st), (g, st)


@pytest.mark.parametrize("s_a", [-128, -60, -54, -30, -24, -23, -22])
@pytest.mark.parametrize("kind,B,N", [("edge", 4, 1000), ("min", 1, 4097), ("edge", 2, 65536), ("max", 3, 2)])
def test_int_ce_loss_grad_extreme_logits(s_a, kind, B, N):
    """Rows of extreme logits, where the low-order Taylor terms carry into
    the bits that decide the rounding (the case that needs the 128-bit
    evaluation)."""
    import torch
    say("loss extreme", s_a, kind, B, N)
    logits = np.full((B, N), 127, np.int8)
    if kind == "edge":
        logits[:, ::3] = -127
    elif kind == "min":
        logits[:, ::2] = -128
    labels = I.labels(610 + N + B, B, N)
    exp, _, st = oracle.int_ce_loss_grad(logits, s_a, labels)
    err = torch.empty((B, N), dtype=torch.int8, device="cuda")
    stats = niti.new_stats()
    ws = niti.new_workspace(niti.workspace_bytes(niti.OP_INT_CE_LOSS, None, B, N))
    niti.int_ce_loss_grad(dev(logits), _i8(s_a), dev(labels), err, stats, ws)
    torch.cuda.synchronize()
    assert (host(err) == exp).all()
    assert same_stats(niti.read_stats(stats)[0], st)


def test_int_ce_loss_worked_examples():
    import json, os, torch
    g = json.load(open(os.path.join(os.path.dirname(__file__), "golden", "loss_examples.json")))
    for c in g["cases"]:
        lg = np.array(c["logits"], np.int8)
        B, N = lg.shape
        err = torch.empty((B, N), dtype=torch.int8, device="cuda")
        stats = niti.new_stats()
        ws = niti.new_workspace(niti.workspace_bytes(niti.OP_INT_CE_LOSS, None, B, N))
        niti.int_ce_loss_grad(dev(lg), _i8(c["s_a"]), dev(np.array(c["labels"], np.int32)), err, stats, ws)
        torch.cuda.synchronize()
        assert host(err).tolist() == c["err"], c["why"]


@pytest.mark.parametrize("n,mu", [(1, 5), (1000, 5), (36864, 3), (2359296, 1), (7, 8),
                                  (1003, 6),        # groups of four plus a 3-weight tail
                                  (4194309, 4)])    # more groups than one pass of the grid covers
def test_sgd_update_parity(n, mu):
    import torch
    say("sgd_update", n, mu)
    w = I.weights(700 + n, (n,))
    g32 = I.uniform_int(800 + n, (n,), -(1 << 26), 1 << 26, dtype=np.int32)
    exp_w, st = oracle.sgd_update(w, g32, mu)
    wd = dev(w)
    stats = niti.new_stats()
    niti.sgd_update(wd, dev(g32), stats, mu)
    torch.cuda.synchronize()
    assert (host(wd) == exp_w).all() and same_stats(niti.read_stats(stats)[0], st)


def test_glue_parity():
    import torch
    say("glue")
    px = I.pixels(5, (3, 3, 10, 12))
    q = oracle.quantize_u8(px)
    x = torch.empty((3, 10, 12, 4), dtype=torch.int8, device="cuda")
    niti.quantize_u8(dev(px), x)
    torch.cuda.synchronize()
    got = nchw(host(x))
    assert (got[:, :3] == q).all() and (got[:, 3] == 0).all()

    a = I.weights(6, (2, 16, 8, 12))
    y_exp, idx_exp = oracle.maxpool2_fwd(a)
    y = torch.empty((2, 4, 6, 16), dtype=torch.int8, device="cuda")
    idx = torch.empty((2, 4, 6, 16), dtype=torch.uint8, device="cuda")
    niti.maxpool2_fwd(dev(nhwc(a)), y, idx)
    torch.cuda.synchronize()
    assert (nchw(host(y)) == y_exp).all() and (nchw(host(idx)) == idx_exp).all()
    dy = I.weights(7, y_exp.shape)
    dx_exp = oracle.maxpool2_bwd(dy, idx_exp, a.shape)
    dx = torch.empty((2, 8, 12, 16), dtype=torch.int8, device="cuda")
    niti.maxpool2_bwd(dev(nhwc(dy)), idx, dx)
    torch.cuda.synchronize()
    assert (nchw(host(dx)) == dx_exp).all()

    e = I.weights(8, (1000,)); act = I.weights(9, (1000,))
    e_exp = oracle.relu_mask(e.copy(), act)
    ed = dev(e)
    niti.relu_mask(ed, dev(act))
    torch.cuda.synchronize()
    assert (host(ed) == e_exp).all()


def test_recorded_calls_replay():
    """Calls recorded once (marshalled arguments) and replayed act like fresh
    calls: the replay reads the buffers' current contents and updates the
    block statistics the same way."""
    import torch
    say("recorded replay")
    M, N, K = 300, 200, 784
    dA = torch.empty((M, K), dtype=torch.int8, device="cuda")
    dB = dev(I.weights(7, (N, K)))
    C = torch.empty((M, N), dtype=torch.int8, device="cuda")
    stats = niti.new_stats()
    sa, sb, sc = _i8(-7), _i8(-9), _i8(0)
    calls = None
    for rep, seed in enumerate([11, 12, 13]):
        A = I.activations(seed, (M, K))
        dA.copy_(dev(A))
        C.fill_(99)
        if calls is None:
            with niti.recording() as calls:
                niti.gemm_fwd(dA, dB, C, stats, sa, sb, sc, 7, True)
            assert len(calls) == 1
        else:
            niti.replay(calls)
        torch.cuda.synchronize()
        exp_out, _, st = oracle.gemm_fwd(A, I.weights(7, (N, K)), relu=True)
        g = niti.read_stats(stats)[0]
        assert (host(C) == exp_out).all(), "rep %d" % rep
        assert same_stats(g, st) and g["calls"] == rep + 1
