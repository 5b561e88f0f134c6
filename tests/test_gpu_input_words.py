"""Input transform and calibration where image rows or pixels start at any byte
address: NCHW widths around the 4- and 8-column words, NHWC channel counts that
are no multiple of four, tensors that end where the last word does.  Against the
CPU oracle, bit for bit."""
import numpy as np
import pytest

import paper_2209_12982_amd as W
import workloads
from oracle import tapwise

from gpu_util import to_device, torch_dev, workspace

pytestmark = pytest.mark.gpu

SHAPES = [(1, 5, 3, 4), (2, 66, 5, 5), (1, 3, 9, 6), (1, 67, 6, 7), (2, 6, 4, 33), (1, 65, 7, 63),
          (1, 10, 5, 65), (1, 7, 2, 66), (1, 4, 5, 3), (1, 9, 1, 1)]


@pytest.mark.parametrize("layout", [W.NCHW, W.NHWC])
@pytest.mark.parametrize("m", [4, 2])
@pytest.mark.parametrize("shape", SHAPES)
def test_input_words(shape, m, layout):
    torch = torch_dev()
    n, cin, h, w = shape
    x, f, b = workloads.random_case(41, n, cin, 8, h, w, signed=True)
    x.reshape(-1)[-3:] = [-128, 127, -128]          # the last bytes count
    ntap = (m + 2) ** 2
    eb = [int(v) for v in np.random.default_rng(42).integers(0, 9, ntap)]
    gp = (W.wino_f4_plan if m == 4 else W.wino_f2_plan)(f, eb, bias=b)
    th, tw = tapwise.tile_grid(h, w, m)
    xd = to_device(x, layout)
    vq = torch.empty((ntap, n * th * tw, cin), dtype=torch.int8, device="cuda")
    W.wino_f4_debug_input_transform(gp, xd, n, h, w, layout, vq, workspace(gp, n, h, w))
    assert (vq.cpu().numpy() == tapwise.input_taps_quantized(x, eb, m=m)).all()
    cal = W.wino_f4_calibrate_input if m == 4 else W.wino_f2_calibrate_input
    e, amax = cal(xd, n, cin, h, w, layout)
    assert amax == tapwise.input_tap_absmax(x, m)
    assert e == tapwise.calibrate_input_exps(x, m=m)


@pytest.mark.parametrize("shape", [(3, 70, 40, 9, 13), (1, 40, 70, 57, 62), (2, 140, 130, 150, 152), (4, 33, 150, 97, 95),
                                   (2, 130, 310, 52, 45)])
@pytest.mark.parametrize("m", [4, 2])
def test_output_maximum(shape, m):
    """calibrate_output on the row-streamed kernel's two block shapes, the
    small-layer kernel's and (F2, last shape) the 64 x 32 blocks: the maximum counts
    in-image outputs only."""
    n, cin, cout, h, w = shape
    x, f, b = workloads.random_case(43, n, cin, cout, h, w, signed=True)
    eb = tapwise.calibrate_input_exps(x, m=m)
    gp = (W.wino_f4_plan if m == 4 else W.wino_f2_plan)(f, eb, bias=b)
    op = tapwise.make_plan(f, eb, bias=b, m=m)
    shift, zmax = W.wino_f4_calibrate_output(gp, to_device(x, W.NHWC), n, h, w, W.NHWC, workspace(gp, n, h, w))
    assert zmax == int(np.abs(tapwise.prequant_output(x, op)).max())
    assert shift == tapwise.calibrate_out_shift(x, op)
