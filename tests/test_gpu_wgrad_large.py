"""Weight gradients of operands whose size is just below 2 GiB: the LDS-staged
kernel's 32-bit offsets run past the last pixel there.  One operand is zero but
for pixels at both ends and at the borders of ranges, so the expected sums are
exact and cheap; the other is full, so any pixel read in the wrong place
shows."""
import numpy as np
import pytest

from paper_2009_13108_amd import niti
from helpers import host, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sparse", ["x", "dy"])
@pytest.mark.parametrize("case", [
    # n, h, w, c, k, r, stride
    (1, (1 << 27) - 1, 1, 16, 16, 1, 1),          # both operands 2 GiB - 16
    (127, 1031, 1025, 16, 16, 1, 1),              # many images
    (3, 6689, 6687, 16, 16, 1, 2),                # the input four times the error
    (1, 26843545, 1, 80, 16, 1, 1),               # plain rows of five 16s
    (5, 2311, 2323, 16, 80, 1, 1),                # the error the larger
])
def test_just_below_two_gigabytes(case, sparse):
    import torch
    n, h, w, c, k, r, stride = case
    say("near 2 GiB", case, sparse)
    d = niti.ConvDesc.make(n, h, w, c, k, r, r, stride, 0)
    npix = n * d.p * d.q
    size = {"x": d.x_shape(), "dy": d.y_shape()}
    gen = torch.Generator(device="cuda").manual_seed(3)
    full = {}
    for name, s in size.items():
        full[name] = torch.empty(s, dtype=torch.int8, device="cuda").random_(-127, 128, generator=gen)
    step = -(-npix // 768)
    at = sorted({0, 1, 63, 64, npix - 1, npix - 2, npix // 2} | {min(npix - 1, i * step) for i in range(0, 768, 37)})
    pix = torch.tensor(at, device="cuda")
    img, rest = pix // (d.p * d.q), pix % (d.p * d.q)
    rows = {"dy": (img, rest // d.q, rest % d.q), "x": (img, rest // d.q * stride, rest % d.q * stride)}
    kept = full[sparse][rows[sparse]].clone()
    full[sparse].zero_()
    full[sparse][rows[sparse]] = kept
    x, dy = (host(full[m][rows[m]]).astype(np.int64) for m in ("x", "dy"))
    exp = dy.T @ x
    w8 = torch.zeros(d.w_shape(), dtype=torch.int8, device="cuda")
    g32 = torch.empty(d.w_shape(), dtype=torch.int32, device="cuda")
    stats = niti.new_stats()
    ws = niti.new_workspace(niti.workspace_bytes(niti.OP_CONV_BWD_WEIGHT, d))
    niti.timing_enable(True)
    niti.conv_bwd_weight(d, full["x"], full["dy"], w8, stats, ws, g32_out=g32, mode=niti.RTN)
    niti.timing_enable(False)
    assert (host(g32).reshape(k, c) == exp).all()
    assert niti.read_stats(stats)[0]["max_abs"] == np.abs(exp).max()
    assert [name for _, name, _ in niti.timing_records() if name.startswith("wgrad")] == [
        "wgrad_dma_kernel<%d,128,4,-2>" % (64 if k <= 64 else 128)]
