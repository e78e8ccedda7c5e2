"""Nine-tap weight gradients with shared rows (3x3, stride 1, padding 1) at the
edges of the scheme: images one row or one or two columns wide, where every
pixel is on a border; rows shorter and longer than the 16 pixels of a lane and
the 128 of a stage; images smaller than a stage, so that one stage holds
several; pixel counts that end inside a stage; several ranges.  The strided and
unpadded layers beside them keep the nine separate runs.  Exact against the
oracle."""
import pytest

import oracle
from paper_2009_13108_amd import inputs as I
from paper_2009_13108_amd import niti
from helpers import dev, host, kcrs, krsc, nhwc, same_stats, say

pytestmark = pytest.mark.gpu

CASES = [
    # n, c, h, w, k, stride, pad
    (3, 64, 1, 1, 64, 1, 1), (5, 64, 1, 40, 64, 1, 1), (7, 64, 33, 1, 64, 1, 1), (9, 64, 5, 2, 128, 1, 1),
    (40, 128, 7, 7, 64, 1, 1), (11, 64, 3, 16, 64, 1, 1), (4, 64, 9, 17, 192, 1, 1), (2, 64, 4, 130, 64, 1, 1),
    (2, 64, 3, 300, 64, 1, 1), (1, 64, 128, 129, 64, 1, 1), (30, 192, 14, 15, 128, 1, 1),
    (3, 64, 9, 9, 64, 1, 0), (3, 64, 9, 9, 64, 2, 1), (2, 64, 8, 8, 64, 1, 2),
]


@pytest.mark.parametrize("case", CASES)
def test_shared_rows(case):
    import torch
    n, c, h, w, k, stride, pad = case
    say("shared rows", case)
    d = oracle.conv_desc(n, c, h, w, k, 3, 3, stride, pad)
    gd = niti.ConvDesc.make(n, h, w, c, k, 3, 3, stride, pad)
    P, Q = oracle.conv_out_hw(d)
    x, wt, dy = I.weights(91, (n, c, h, w)), I.weights(92, (k, c, 3, 3)), I.errors8(93, (n, k, P, Q))
    exp_w, exp_g, st = oracle.conv_bwd_weight(d, x, dy, wt, mu=5)
    ws = niti.new_workspace(niti.workspace_bytes(niti.OP_CONV_BWD_WEIGHT, gd))
    g32 = torch.empty(gd.w_shape(), dtype=torch.int32, device="cuda")
    stats = niti.new_stats()
    wd = dev(krsc(wt))
    niti.conv_bwd_weight(gd, dev(nhwc(x)), dev(nhwc(dy)), wd, stats, ws, g32_out=g32, mu=5)
    assert (kcrs(host(g32)) == exp_g).all()
    assert (kcrs(host(wd)) == exp_w).all() and same_stats(niti.read_stats(stats)[0], st)
