"""The passes beside the contractions at the edges of their vector forms:
channel counts that fill 16-byte pieces, only 4-byte words, or neither;
tensors at addresses that allow wide accesses and views that do not; element
counts around a piece, a workgroup's share and the grid's limit.  All results
are integers, so every comparison with the oracle is exact."""
import numpy as np
import pytest

import oracle
from paper_2009_13108_amd import inputs as I
from paper_2009_13108_amd import niti
from helpers import host, nchw, nhwc, say, same_stats

pytestmark = pytest.mark.gpu


def placed(a, shift):
    """a on the device, `shift` bytes past a 16-byte boundary."""
    import torch
    flat = torch.from_numpy(np.ascontiguousarray(a)).view(torch.uint8).reshape(-1)
    buf = torch.empty(flat.numel() + 16, dtype=torch.uint8, device="cuda")
    t = buf[shift:shift + flat.numel()]
    t.copy_(flat)
    return t.view(torch.int8 if a.dtype == np.int8 else torch.uint8).view(a.shape)


POOL = [(1, 2, 2, 1), (3, 6, 10, 3), (2, 4, 6, 4), (3, 10, 14, 20), (2, 8, 12, 16), (5, 14, 2, 48), (64, 64, 64, 32)]


@pytest.mark.parametrize("shape", POOL)
@pytest.mark.parametrize("shift", [0, 4, 1])
def test_pooling_forms(shape, shift):
    n, h, w, c = shape
    say("pool", shape, shift)
    a = I.weights(21, (n, c, h, w))
    a.reshape(-1)[::3] = -128                 # the type's lowest value, and many ties
    a.reshape(-1)[1::7] = 127
    y_exp, i_exp = oracle.maxpool2_fwd(a)
    dy = I.weights(22, y_exp.shape)
    dx_exp = oracle.maxpool2_bwd(dy, i_exp, a.shape)
    x = placed(nhwc(a), shift)
    y, idx, dx = (placed(np.full(s, 99, t), shift) for s, t in
                  (((n, h // 2, w // 2, c), np.int8), ((n, h // 2, w // 2, c), np.uint8), ((n, h, w, c), np.int8)))
    niti.maxpool2_fwd(x, y, idx)
    niti.maxpool2_bwd(placed(nhwc(dy), shift), idx, dx)
    assert (nchw(host(y)) == y_exp).all() and (nchw(host(idx)) == i_exp).all()
    assert (nchw(host(dx)) == dx_exp).all()


@pytest.mark.parametrize("case", [(2, 3, 5, 7, 4, 0), (3, 3, 6, 10, 4, 0), (2, 1, 28, 28, 4, 0), (2, 4, 8, 8, 4, 0),
                                  (2, 3, 8, 8, 4, 4), (2, 3, 8, 8, 8, 0), (7, 2, 32, 36, 4, 0)])
def test_quantisation_forms(case):
    n, c, h, w, cp, shift = case
    say("quantize", case)
    px = I.pixels(23, (n, c, h, w))
    x = placed(np.full((n, h, w, cp), 99, np.int8), shift)
    niti.quantize_u8(placed(px, 0), x)
    got = nchw(host(x))
    assert (got[:, :c] == oracle.quantize_u8(px)).all() and (got[:, c:] == 0).all()


@pytest.mark.parametrize("n", [1, 15, 16, 17, 4095, 4096 * 16 + 5, 4096 * 256 * 16 + 33])
@pytest.mark.parametrize("shift", [0, 1])
def test_mask_and_dropout_forms(n, shift):
    say("mask and dropout", n, shift)
    e, act = I.weights(24, (n,)), I.weights(25, (n,))
    act[::5] = 0
    act[1::9] = -128
    ed = placed(e, shift)
    niti.relu_mask(ed, placed(act, shift))
    assert (host(ed) == np.where(act > 0, e, 0)).all()
    y_exp, k_exp = oracle.dropout_fwd(e, 31, 2, 128)[:2]
    y, keep, dx = (placed(np.full(n, 99, t), shift) for t in (np.int8, np.uint8, np.int8))
    niti.dropout_fwd(placed(e, shift), y, keep, 31, 2, 128)
    niti.dropout_bwd(placed(act, shift), keep, dx)
    assert (host(y) == y_exp).all() and (host(keep) == k_exp).all()
    assert (host(dx) == np.where(k_exp != 0, act, 0)).all()


@pytest.mark.parametrize("n", [1, 3, 4, 5, 1023, 8192 * 4 + 2, 512 * 256 * 16 + 7])
@pytest.mark.parametrize("mode", [oracle.PSR, oracle.RTN, oracle.SR])
def test_int32_passes_forms(n, mode):
    """The maximum in the first, the last and a ragged element."""
    import torch
    say("int32 passes", n, mode)
    g = I.uniform_int(26, (n,), -50000, 50000, dtype=np.int32)
    for at in {0, n - 1, n // 2}:
        x = g.copy()
        x[at] = -(2 ** 31)
        exp, st = oracle.shift_round(x, 7, mode)
        stats = niti.new_stats()
        y = torch.empty(n, dtype=torch.int8, device="cuda")
        xd = torch.from_numpy(x).cuda()
        niti.round_psr(xd, y, -1, 7, stats, mode=mode)
        assert (host(y) == exp).all() and same_stats(niti.read_stats(stats)[0], st)
