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
