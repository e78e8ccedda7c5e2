"""Splits of the weight-gradient reduction, seen through the workspace sizes
(which need no GPU)."""
import pytest

from paper_2009_13108_amd import niti


def splits(d):
    """The pixel ranges that the workspace of niti_conv_bwd_weight holds."""
    nw = d.k * d.r * d.s * d.c * 4
    up = (nw + 255) // 256 * 256
    rest = niti.workspace_bytes(niti.OP_CONV_BWD_WEIGHT, d) - up
    return max(1, rest // nw)


@pytest.mark.parametrize("c, k", [(64, 64), (64, 192), (64, 384), (128, 256), (192, 256), (320, 128), (256, 320),
                                  (320, 512), (512, 512)])
@pytest.mark.parametrize("h, stride, pad", [(7, 2, 1), (14, 2, 1), (28, 2, 1), (56, 2, 1), (28, 1, 0), (28, 1, 1)])
def test_nine_run_weight_gradient_fills_one_round(c, k, h, stride, pad):
    """3 x 3 layers that are not read in shared rows: a workgroup holds its CU,
    so more than 256 of them take a second round (up to 1.7 times as long);
    short ranges (under 13 stages) lose more in partial sums than they gain
    from the last quarter of the CUs."""
    for n in (1, 2, 4, 8, 16, 32, 64, 100, 128, 256):
        if n * h * h * max(c, k) > 1 << 28 or (stride == 1 and pad == 1 and c >= 128):
            continue
        d = niti.ConvDesc.make(n, h, h, c, k, 3, 3, stride, pad)
        tiles = (c // 32) * (k // 64)
        stages = -(-n * d.p * d.q // 128)
        got = splits(d)
        low = min(-(-192 // tiles), max(1, stages // 2))     # three quarters of the CUs
        low = -(-stages // -(-stages // low))
        assert got == low or tiles * got <= 256, n
        if got > low:
            assert -(-stages // got) >= 13, n


def test_near_two_gigabytes_keeps_the_lds_kernel():
    """Operands whose size is just below 2 GiB: the plan of the LDS-staged
    kernel (ranges for three workgroups per CU), as for smaller ones."""
    d = niti.ConvDesc.make(1, (1 << 27) - 1, 1, 16, 16, 1, 1, 1, 0)
    assert splits(d) == 768
