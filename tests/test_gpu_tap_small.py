"""The small-layer kernels (one wave per row of taps) against the CPU oracle, bit
for bit: the tap GEMM behind the input transform, and the convolution in one
launch; each of their block shapes at ragged tile and channel counts, one and
several 64-channel chunks, channel blocks that leave a partial group, both
transforms and layouts."""
import numpy as np
import pytest

import paper_2209_12982_amd as W
import workloads
from oracle import tapwise

from gpu_util import empty_out, from_device_nchw, run_conv, to_device, torch_dev, workspace

pytestmark = pytest.mark.gpu

# n, cin, cout, tile rows, tile columns, cut (pixels the last tile lacks); the
# block counts on 256 compute units select 32x32, 16x32 and 16x16 blocks
SHAPES = [
    (4, 70, 130, 17, 16, 1),     # 34 tile blocks of 32 x 5 channel blocks of 32
    (3, 64, 150, 12, 16, 0),     # 18 x 10 channel blocks of 16, one chunk
    (1, 200, 36, 5, 7, 1),       # 3 x 3 blocks of 16, four chunks
    (1, 5, 300, 1, 3, 1),        # a single tile block, 19 channel blocks
]
BLOCKS = [(32, 32), (16, 32), (16, 16), (16, 16)]


@pytest.mark.parametrize("layout", [W.NCHW, W.NHWC])
@pytest.mark.parametrize("m", [4, 2])
@pytest.mark.parametrize("shape", SHAPES)
def test_small_tap_gemm(shape, m, layout):
    torch = torch_dev()
    n, cin, cout, th, tw, cut = shape
    h, w = m * th - cut, m * tw - cut
    x, f, b = workloads.random_case(31, n, cin, cout, h, w, signed=True)
    spec = tapwise.F4 if m == 4 else tapwise.F2
    eb = tapwise.calibrate_input_exps(x, m=m)
    relu = cut == 1
    op = tapwise.make_plan(f, eb, bias=b, out_shift=10, relu=relu, m=m)
    gp = (W.wino_f4_plan if m == 4 else W.wino_f2_plan)(f, eb, bias=b, out_shift=10, relu=relu)
    assert W.wino_f4_plan_info(gp)["epilogue_bits"] == 32 and spec.m == m
    assert W.wino_f4_tap_kernel_choice(gp, n, h, w) == W.TAP_RESIDENT_64X32
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        k = W.wino_probe_conv_kernels(gp, 1, n, h, w, layout)       # an odd address: never the one launch
        assert (k["launches"], k["gemm"], k["co"], k["tiles"]) == (2, "small", *BLOCKS[SHAPES.index(shape)]), k
    xd, y, ws = to_device(x, layout), empty_out(n, cout, h, w, layout), workspace(gp, n, h, w)
    W.wino_f4_input_transform(gp, xd, n, h, w, layout, ws)
    W.wino_f4_tap_gemm(gp, ws, y, n, h, w, layout)
    ref = tapwise.conv_int8(x, op)
    got = from_device_nchw(y, layout)
    assert (got == ref).all(), f"tap GEMM: {(got != ref).sum()} mismatches"
    got = run_conv(gp, x, layout)
    assert (got == ref).all(), f"convolution: {(got != ref).sum()} mismatches"


# n, cin, cout, h, w, whether a tap's e_B lies past the one-instruction form, and
# on 256 compute units the block's channels in the one launch by (transform,
# layout), 0 for two launches: words shifted inside pixels and rows, the image's
# last bytes, both requantization forms at every block width, up to four chunks
F4N, F4C, F2N, F2C = (4, W.NCHW), (4, W.NHWC), (2, W.NCHW), (2, W.NHWC)
ONE_LAUNCH = [
    (10, 5, 50, 31, 32, False, {F2N: 64, F2C: 64}),
    (10, 5, 50, 31, 32, True, {F2N: 64, F2C: 64}),
    (2, 70, 200, 27, 28, False, {F2N: 32, F2C: 32}),
    (2, 70, 200, 27, 28, True, {F2N: 32, F2C: 32}),
    (2, 130, 200, 27, 28, False, {F2C: 32}),
    (1, 200, 20, 4, 4, False, {F2C: 16}),
    (1, 66, 20, 9, 8, True, {F2N: 16, F2C: 16, F4C: 16}),
    (1, 67, 33, 13, 5, True, {F2N: 16, F2C: 16, F4C: 16}),
    (1, 35, 33, 13, 5, True, {F2N: 16, F2C: 16, F4N: 16, F4C: 16}),
    (3, 64, 16, 6, 7, False, {F2N: 16, F2C: 16, F4N: 16, F4C: 16}),
    (1, 3, 9, 9, 3, False, {F2N: 0, F2C: 0, F4N: 0, F4C: 0}),     # below four channels (NHWC) or columns (NCHW)
]


@pytest.mark.parametrize("layout", [W.NCHW, W.NHWC])
@pytest.mark.parametrize("m", [4, 2])
@pytest.mark.parametrize("shape", ONE_LAUNCH)
def test_one_launch_convolution(shape, m, layout):
    torch = torch_dev()
    n, cin, cout, h, w, past, kernel = shape
    x, f, b = workloads.random_case(33, n, cin, cout, h, w, signed=True)
    x.reshape(-1)[-3:] = [-128, 127, -128]
    eb = tapwise.calibrate_input_exps(x, m=m)
    eg = tapwise.make_plan(f, eb, m=m)["e_g"]
    if past:
        # one tap beyond e_B = 8 sends every tap through the shift-and-clamp form;
        # its e_G falls as far, which leaves the alignment shifts as they were
        t = len(eb) // 2
        eg[t] -= 9 - eb[t]
        eb[t] = 9
    op = tapwise.make_plan(f, eb, e_g=eg, bias=b, out_shift=9, relu=past, m=m)
    gp = (W.wino_f4_plan if m == 4 else W.wino_f2_plan)(f, eb, w_exp=eg, bias=b, out_shift=9, relu=past)
    assert W.wino_f4_plan_info(gp)["epilogue_bits"] == 32 and (max(eb) > 8) == past
    if torch.cuda.get_device_properties(0).multi_processor_count == 256 and (m, layout) in kernel:
        k = W.wino_probe_conv_kernels(gp, 0, n, h, w, layout)
        assert (k["co"] if k["launches"] == 1 else 0) == kernel[(m, layout)], k
    vq = tapwise.input_taps_quantized(x, eb, m=m)
    assert (vq.reshape(len(eb), -1) != 0).any(axis=1).all()       # every tap counts
    y = run_conv(gp, x, layout)
    ref = tapwise.conv_int8(x, op)
    assert (y == ref).all(), f"{(y != ref).sum()} mismatches"


@pytest.mark.parametrize("layout", [W.NCHW, W.NHWC])
@pytest.mark.parametrize("m", [4, 2])
def test_output_over_the_input(m, layout):
    """A layer of the one launch's sizes whose output overlaps its input, wholly or in
    part: two launches, which read x before they write y, as before that kernel."""
    torch = torch_dev()
    n, c, h, w = 4, 48, 24, 28
    x, f, b = workloads.random_case(35, n, c, c, h, w, signed=True)
    eb = tapwise.calibrate_input_exps(x, m=m)
    op = tapwise.make_plan(f, eb, bias=b, out_shift=9, m=m)
    gp = (W.wino_f4_plan if m == 4 else W.wino_f2_plan)(f, eb, bias=b, out_shift=9)
    xd, ref = to_device(x, layout).reshape(-1), tapwise.conv_int8(x, op)
    ws = workspace(gp, n, h, w)
    for off in (0, 4, xd.numel() - 4):
        buf = torch.zeros(xd.numel() + off, dtype=torch.int8, device="cuda")
        buf[:xd.numel()] = xd
        assert W.wino_probe_conv_kernels(gp, buf, n, h, w, layout)["launches"] == 1
        W.wino_f4_conv_int8(gp, buf[:xd.numel()], buf[off:], n, h, w, layout, W.SPLIT, ws)
        y = buf[off:].reshape((n, c, h, w) if layout == W.NCHW else (n, h, w, c))
        assert (from_device_nchw(y, layout) == ref).all(), off


def test_f2_wide_blocks():
    """The F2 sizes that keep the 64x32 tap-resident blocks under AUTO."""
    torch = torch_dev()
    n, cin, cout, h, w = 8, 200, 510, 20, 20
    x, f, b = workloads.random_case(34, n, cin, cout, h, w, signed=True)
    eb = tapwise.calibrate_input_exps(x, m=2)
    op = tapwise.make_plan(f, eb, bias=b, out_shift=10, m=2)
    gp = W.wino_f2_plan(f, eb, bias=b, out_shift=10)
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        k = W.wino_probe_conv_kernels(gp, 0, n, h, w, W.NHWC)
        assert (k["gemm"], k["co"], k["tiles"]) == ("resident", 64, 32), k
    for layout in (W.NCHW, W.NHWC):
        assert (run_conv(gp, x, layout) == tapwise.conv_int8(x, op)).all()


@pytest.mark.parametrize("layout", [W.NCHW, W.NHWC])
def test_small_tap_gemm_unaligned_output(layout):
    """An output that is not 4-byte aligned takes the byte stores."""
    torch = torch_dev()
    n, cin, cout, h, w = 1, 32, 64, 8, 8
    x, f, b = workloads.random_case(32, n, cin, cout, h, w, signed=True)
    for m, plan in ((4, W.wino_f4_plan), (2, W.wino_f2_plan)):
        eb = tapwise.calibrate_input_exps(x, m=m)
        gp = plan(f, eb, bias=b, out_shift=9)
        op = tapwise.make_plan(f, eb, bias=b, out_shift=9, m=m)
        xa = np.ascontiguousarray(x if layout == W.NCHW else x.transpose(0, 2, 3, 1))
        buf = torch.full((n * cout * h * w + 1,), 77, dtype=torch.int8, device="cuda")
        ws = torch.empty(W.wino_f4_workspace_bytes(gp, n, h, w), dtype=torch.int8, device="cuda")
        W.wino_f4_conv_int8(gp, torch.from_numpy(xa).cuda(), buf[1:], n, h, w, layout, W.SPLIT, ws)
        got = buf.cpu().numpy()
        assert got[0] == 77
        ref = tapwise.conv_int8(x, op)
        ref = ref if layout == W.NCHW else ref.transpose(0, 2, 3, 1)
        assert (got[1:] == ref.reshape(-1)).all()
