"""The rules that pick a convolution's kernels, at sizes either side of their
lines: layers that were measured slower on the other side.  Which kernels run is
asked of the library (host only); every pair of sides is compared with the oracle
elsewhere, and here where a rule sends a form to a kernel it had not reached."""
import numpy as np
import pytest

import paper_2209_12982_amd as W
import workloads
from oracle import tapwise

from gpu_util import run_conv, torch_dev

pytestmark = pytest.mark.gpu


def _kernels(m, n, cin, cout, h, w, layout, epi=32):
    torch = torch_dev()
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the sizes below are for 256 compute units")
    f = torch.randn((cout, cin, 3, 3), device="cuda", generator=torch.Generator("cuda").manual_seed(51)) * 0.02
    x = (torch.randn((1, 16, 48, 48), device="cuda", generator=torch.Generator("cuda").manual_seed(52)) * 24).clamp_(
        0, 127).to(torch.int8)
    eb, _ = (W.wino_f4_calibrate_input if m == 4 else W.wino_f2_calibrate_input)(x, 1, 16, 48, 48, W.NCHW)
    plan = (W.wino_f4_plan_device if m == 4 else W.wino_f2_plan_device)(f, eb)
    assert epi is None or W.wino_f4_plan_info(plan)["epilogue_bits"] == epi
    return W.wino_probe_conv_kernels(plan, 0, n, h, w, layout)


# NCHW band transform: tiles per block (16 are faster by a tenth to a quarter
# where 8 would leave only a few idle tiles less in a row)
@pytest.mark.parametrize("m,n,cin,h,w,tiles", [
    (4, 8, 256, 227, 196, 16), (4, 8, 64, 283, 208, 16), (4, 4, 128, 408, 392, 16), (4, 8, 512, 196, 136, 16),
    (4, 2, 256, 75, 75, 8), (4, 8, 512, 33, 66, 8), (4, 2, 128, 183, 144, 8), (4, 1, 64, 568, 568, 16),
    (2, 8, 128, 189, 208, 16), (2, 1, 64, 343, 204, 16), (2, 8, 512, 29, 38, 8),
])
def test_band_transform_width(m, n, cin, h, w, tiles):
    k = _kernels(m, n, cin, 512, h, w, W.NCHW, epi=None)
    assert (k["launches"], k["xform"], k["xform_tiles"]) == (2, "band", tiles), k


# The one launch, 0 for two launches, else its block's channels
@pytest.mark.parametrize("m,layout,n,cin,cout,h,w,co", [
    (2, W.NCHW, 1, 16, 16, 32, 32, 16), (2, W.NCHW, 8, 64, 64, 56, 56, 64),
    (2, W.NCHW, 1, 64, 384, 94, 64, 0), (2, W.NCHW, 8, 64, 512, 28, 28, 0), (2, W.NCHW, 1, 32, 32, 196, 249, 64),
    (2, W.NCHW, 1, 128, 128, 47, 39, 16), (2, W.NCHW, 1, 128, 128, 112, 112, 0), (2, W.NCHW, 4, 128, 64, 64, 80, 0),
    (2, W.NCHW, 1, 96, 64, 169, 163, 64), (2, W.NCHW, 2, 192, 192, 42, 36, 0), (2, W.NCHW, 1, 512, 64, 28, 28, 0),
    (2, W.NHWC, 8, 64, 64, 56, 56, 64), (2, W.NHWC, 8, 256, 256, 14, 14, 32), (2, W.NHWC, 1, 320, 64, 14, 14, 16),
    (2, W.NHWC, 2, 384, 384, 25, 33, 64), (2, W.NHWC, 1, 384, 64, 14, 14, 0), (2, W.NHWC, 1, 512, 64, 14, 14, 0),
    (4, W.NHWC, 8, 128, 128, 32, 32, 16), (4, W.NHWC, 1, 192, 64, 28, 28, 0),
    (4, W.NCHW, 1, 64, 64, 28, 28, 16), (4, W.NCHW, 8, 128, 128, 32, 32, 0), (4, W.NCHW, 1, 96, 64, 28, 28, 0),
])
def test_one_launch(m, layout, n, cin, cout, h, w, co):
    k = _kernels(m, n, cin, cout, h, w, layout)
    assert (k["co"] if k["launches"] == 1 else 0) == co, k


# F2 tap GEMM of two launches: the tap-resident kernel's 64 x 32 blocks or the
# small-layer kernel
@pytest.mark.parametrize("n,cin,cout,h,w,gemm", [
    (2, 192, 320, 52, 46, "resident"), (8, 192, 384, 20, 28, "resident"), (1, 256, 128, 118, 90, "resident"),
    (1, 192, 192, 85, 85, "resident"), (1, 64, 512, 112, 112, "small"), (1, 256, 256, 112, 112, "small"),
    (8, 512, 512, 25, 33, "resident"), (1, 320, 384, 96, 96, "resident"), (1, 256, 256, 126, 112, "small"),
    (1, 512, 128, 198, 140, "small"), (1, 512, 512, 64, 80, "small"),
    (4, 320, 48, 173, 249, "resident"), (2, 192, 64, 487, 360, "resident"), (8, 256, 64, 175, 125, "small"),
    (8, 128, 128, 309, 210, "small"), (4, 256, 32, 310, 433, "small"),
])
def test_f2_tap_gemm(n, cin, cout, h, w, gemm):
    for layout in (W.NCHW, W.NHWC):
        k = _kernels(2, n, cin, cout, h, w, layout, epi=None if cin > 256 else 32)
        assert (k["launches"], k["gemm"]) == (2, gemm), k


# F4 tap GEMM of two launches: the small-layer kernel while its 32 x 32 blocks run
# at once, then the row-streamed one
@pytest.mark.parametrize("n,cin,cout,h,w,gemm", [
    (1, 96, 320, 134, 118, "rows"), (2, 64, 256, 76, 120, "rows"), (1, 128, 256, 131, 127, "rows"),
    (1, 256, 32, 467, 300, "rows"), (1, 64, 64, 568, 568, "rows"), (4, 256, 256, 160, 160, "rows"),
    (1, 64, 256, 116, 109, "small"), (1, 256, 256, 129, 124, "small"), (4, 256, 32, 150, 202, "small"),
    (2, 256, 256, 75, 75, "small"), (8, 256, 512, 32, 32, "small"),
])
def test_f4_tap_gemm(n, cin, cout, h, w, gemm):
    for layout in (W.NCHW, W.NHWC):
        k = _kernels(4, n, cin, cout, h, w, layout)
        assert (k["launches"], k["gemm"]) == (2, gemm), k


@pytest.mark.parametrize("layout", [W.NCHW, W.NHWC])
def test_small_kernel_on_many_narrow_blocks(layout):
    """Few output channels, as many 64 x 64 blocks as used to go to the
    row-streamed kernel: the small-layer kernel's 32 x 32 blocks at one per
    compute unit, ragged in channels and tiles."""
    torch_dev()
    n, cin, cout, h, w = 3, 70, 27, 207, 201
    x, f, b = workloads.random_case(53, n, cin, cout, h, w, signed=True)
    eb = tapwise.calibrate_input_exps(x, m=4)
    op = tapwise.make_plan(f, eb, bias=b, out_shift=10, relu=True, m=4)
    gp = W.wino_f4_plan(f, eb, bias=b, out_shift=10, relu=True)
    k = W.wino_probe_conv_kernels(gp, 0, n, h, w, layout)
    assert (k["gemm"], k["co"], k["tiles"]) == ("small", 32, 32), k
    assert (run_conv(gp, x, layout) == tapwise.conv_int8(x, op)).all()
