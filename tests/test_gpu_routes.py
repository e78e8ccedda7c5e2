"""Which kernel a call runs, read from the library's timing records, on both
sides of each rule that chooses by size.  The results are exact whichever
kernel runs (the parity tests compare them at these sizes and others); these
cases keep a rule from moving over shapes where its kernel is the slower one."""
import pytest

from paper_2009_13108_amd import niti
from helpers import say

pytestmark = pytest.mark.gpu


def kernels(call):
    """Labels of the contraction launches and split sums of one call."""
    import torch
    niti.timing_enable(True)
    call()
    niti.timing_enable(False)
    torch.cuda.synchronize()
    return [name for fam, name, _ in niti.timing_records() if fam in (niti.TIMING_KERNEL, niti.TIMING_SUM)]


def i8(*shape):
    import torch
    return torch.ones(shape, dtype=torch.int8, device="cuda")


def run_gemm(M, N, K, mode=niti.PSR):
    return kernels(lambda: niti.gemm_fwd(i8(M, K), i8(N, K), i8(M, N), niti.new_stats(), mode=mode))


def run_conv(op, n, h, c, k, r, stride, pad, mode=niti.PSR):
    d = niti.ConvDesc.make(n, h, h, c, k, r, r, stride, pad)
    x, w, y, stats = i8(*d.x_shape()), i8(*d.w_shape()), i8(*d.y_shape()), niti.new_stats()
    ws = niti.new_workspace(niti.workspace_bytes(
        {"fwd": niti.OP_CONV_FWD, "bwd": niti.OP_CONV_BWD_DATA, "wgrad": niti.OP_CONV_BWD_WEIGHT}[op], d))
    if op == "fwd":
        return kernels(lambda: niti.conv_fwd(d, x, w, y, stats, mode=mode, ws=ws))
    if op == "bwd":
        return kernels(lambda: niti.conv_bwd_data(d, y, w, x, stats, ws, mode=mode))
    return kernels(lambda: niti.conv_bwd_weight(d, x, y, w, stats, ws, mode=mode))


GATHERED = ["wgrad_small_kernel<-1>", "wgrad_small_kernel<0>"]
TWICE = ["wgrad_dma_kernel<128,128,3,-1>", "wgrad_dma_kernel<128,128,3,0>"]
STORED = ["wgrad_dma_kernel<128,128,4,-2>", "split_sum<1>"]


@pytest.mark.parametrize("case", [
    # n, h, c, k, r, stride, pad, mode, launches
    (64, 1, 512, 512, 1, 1, 0, niti.PSR, GATHERED),       # 256 tiles of 32 x 32
    (64, 1, 528, 512, 1, 1, 0, niti.PSR, TWICE),          # 272
    (32, 1, 1024, 1024, 1, 1, 0, niti.PSR, TWICE),
    (1000, 1, 640, 640, 1, 1, 0, niti.PSR, None),         # 400, more samples than the twice form takes
    (12, 1, 2720, 166, 1, 1, 0, niti.PSR, GATHERED),      # rows the LDS kernel does not take: 510 tiles
    (12, 1, 3656, 167, 1, 1, 0, niti.PSR, ["wgrad_kernel<128,128>", "split_sum<1>"]),   # 690 tiles
    (128, 1, 3656, 167, 1, 1, 0, niti.PSR, GATHERED),
], ids=str)
def test_gathered_weight_gradient(case):
    say("gathered", case)
    got = run_conv("wgrad", *case[:8])
    if case[8] is None:
        assert not [g for g in got if g.startswith("wgrad_small_kernel")], got
    else:
        assert got == case[8]


@pytest.mark.parametrize("case", [
    (16, 1, 1056, 1008, 1, 1, 0, niti.PSR, TWICE),
    (16, 1, 1056, 1008, 1, 1, 0, niti.SR, [TWICE[0], "wgrad_dma_kernel<128,128,3,2>"]),
    (8, 13, 32, 192, 5, 2, 2, niti.SR, STORED),           # 153600 weights, 392 pixels
    (8, 13, 32, 192, 5, 2, 2, niti.PSR, STORED),
    (1, 13, 32, 192, 5, 2, 2, niti.PSR, TWICE),           # 49 pixels
    (1, 13, 32, 192, 5, 2, 2, niti.SR, STORED),
    (16, 1, 16400, 32, 1, 1, 0, niti.PSR, ["wgrad_dma_kernel<64,128,4,-2>", "split_sum<1>"]),
    (16, 1, 16400, 48, 1, 1, 0, niti.PSR, ["wgrad_dma_kernel<64,128,3,-1>", "wgrad_dma_kernel<64,128,3,0>"]),
], ids=str)
def test_weight_gradient_formed_twice(case):
    say("twice", case)
    assert run_conv("wgrad", *case[:8]) == case[8]


@pytest.mark.parametrize("case", [
    (64, 4096, 4096, ["igemm_small_main<1,2>"]),           # 256 tiles of 32 rows: one per CU
    (33, 4128, 256, ["igemm_small_main<1,4>"]),            # 258
    (44, 6541, 1844, ["igemm_small_main<0,4>"]),
    (32, 8000, 256, ["igemm_small_main<1,2>"]),            # no second 32 rows
    (84, 4688, 2048, ["igemm_small_main<1,4>"]),           # 441 of 32 rows, 294 of 64: one batch of loads,
    (84, 4688, 2064, ["igemm_small_main<1,2>"]),           # and more
    (84, 4688, 1023, ["igemm_small_main<0,4>"]),
    (84, 4688, 1025, ["igemm_small_main<0,2>"]),
    (84, 4096, 4096, ["igemm_small_main<1,4>"]),           # 256 of 64 rows
], ids=str)
def test_small_product_rows(case):
    say("small product", case)
    assert run_gemm(*case[:3]) == case[3]


@pytest.mark.parametrize("case", [
    (40000, 48, 1024, "256,64,4,8,1,64"),
    (4096, 1100, 64, "128,128,4,4,2,64"),        # 288 tiles: one step,
    (4096, 1100, 368, "128,128,4,4,2,64"),       # a short reduction,
    (4096, 1100, 384, "128,128,2,4,2,128"),
    (4096, 1100, 1088, "128,128,2,4,2,128"),
    (3072, 1100, 1152, "128,128,4,4,2,64"),      # 216 tiles
    (4096, 2176, 1088, "128,128,4,4,2,64"),      # 544: the second round leaves most CUs one; odd multiple of 64
    (4096, 2176, 1152, "128,128,2,4,2,128"),
    (16384, 2100, 752, "128,128,4,4,2,64"),      # 2176 tiles
    (16384, 2100, 768, "128,128,2,4,2,128"),
    (16384, 2100, 1072, "128,128,4,4,2,64"),     # the last step is half empty
    (16500, 1900, 1552, "128,128,2,4,2,128"),
    (16384, 1024, 624, "256,256,3,2,4,64"),      # tiles of 256
    (16384, 1024, 640, "256,256,2,2,4,128"),
    (16384, 1024, 1072, "256,256,3,2,4,64"),
    (16384, 1024, 2096, "256,256,2,2,4,128"),
    (16384, 1024, 2112, "256,256,3,2,4,64"),     # odd multiple of 64
    (12800, 1100, 384, "256,256,3,2,4,64"),      # a round of 256 (padded) against two of 128
    (42000, 320, 320, "128,128,4,4,2,64"),       # two against two
    (16384, 2100, 1136, "128,128,2,4,2,128"),    # three against five, short
    (16384, 2100, 1152, "256,256,2,2,4,128"),    # and longer
], ids=str)
def test_ring_steps(case):
    say("ring steps", case)
    assert run_gemm(*case[:3]) == ["igemm_dma_main<%s,0>" % case[3]]


@pytest.mark.parametrize("case", [
    ("fwd", 60, 28, 128, 256, 1, 1, 0, "128,128,4,4,2,64"),     # 368 x 2 tiles, 128 products per output
    ("fwd", 60, 28, 128, 160, 3, 1, 1, "128,128,4,4,2,64"),     # 736: the second round leaves most CUs one
    ("fwd", 70, 28, 128, 160, 3, 1, 1, "128,128,2,4,2,128"),    # 858
    ("fwd", 128, 14, 256, 160, 3, 1, 1, "128,128,2,4,2,128"),   # 392
    ("fwd", 120, 14, 128, 160, 3, 1, 1, "128,128,4,4,2,64"),    # 368: short, few CUs with two workgroups
    ("fwd", 128, 14, 128, 160, 3, 1, 1, "128,128,2,4,2,128"),
    ("fwd", 80, 28, 512, 256, 1, 1, 0, "256,256,3,2,4,64"),
    ("fwd", 80, 28, 1152, 256, 1, 1, 0, "256,256,3,2,4,64"),
    ("fwd", 80, 28, 2048, 256, 1, 1, 0, "256,256,2,2,4,128"),
    ("fwd", 60, 28, 192, 160, 3, 1, 1, "128,128,4,4,2,64"),     # channels that are not whole 128s
], ids=str)
def test_ring_steps_of_convolutions(case):
    say("ring steps", case)
    assert run_conv(*case[:8]) == ["igemm_dma_main<%s,1>" % case[8]]


@pytest.mark.parametrize("case", [
    ("fwd", 1, 14, 32, 20, 3, 1, 1, "igemm_main"),        # 288 products per output, 20 channels
    ("fwd", 1, 14, 48, 20, 3, 1, 1, "igemm_dma_main"),    # 432
    ("fwd", 1, 14, 48, 10, 3, 1, 1, "igemm_main"),
    ("fwd", 1, 14, 80, 10, 3, 1, 1, "igemm_dma_main"),    # 720
    ("fwd", 1, 14, 32, 32, 3, 1, 1, "igemm_dma_main"),
    ("bwd", 1, 32, 16, 16, 3, 2, 1, "igemm_main"),        # 16 channels
    ("bwd", 1, 56, 36, 48, 3, 2, 1, "igemm_main"),
    ("bwd", 60, 56, 36, 48, 3, 2, 1, "igemm_dma_main"),   # 1472 tiles
], ids=str)
def test_carried_pieces(case):
    say("carried pieces", case)
    got = run_conv(*case[:8])
    assert len(got) == 1 and got[0].split("<")[0] == case[8], got


@pytest.mark.parametrize("case", [
    (100, 100, 65, niti.SR, ["igemm_main<64,64,1>"]),
    (100, 100, 200, niti.SR, ["igemm_main<64,64,4>"]),
    (2600, 1030, 65, niti.SR, ["igemm_main<64,64,4>"]),   # 189 tiles of 128
    (5000, 1030, 65, niti.SR, ["igemm_main<128,128,1>"]),
], ids=str)
def test_general_kernel_lookahead(case):
    say("look-ahead", case)
    assert run_gemm(*case[:4]) == case[4]
