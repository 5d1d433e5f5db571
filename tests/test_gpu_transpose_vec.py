"""Column-major copies of planes beyond LDS, by 16-byte vectors where rows and
columns are whole vectors (else element by element, the last case): tiles of
64 x 64 whole and cut at both edges, against the oracle."""
import pytest
import torch

import workloads
from gpu_util import FP32_TOL, assert_close, dev, log, to_f64, upload_f32, upload_stream
from paper_2412_16602_amd import vmb
from test_gpu_cross import test_cross_merge_bit_exact as merge_bit_exact
from test_gpu_scan import merged_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W,dtype", [(128, 128, "f32"), (68, 196, "f32"), (260, 60, "f32"),
                                       (128, 128, "bf16"), (72, 200, "bf16"), (264, 56, "bf16"),
                                       (132, 100, "bf16")])
def test_transpose_vec(H, W, dtype):
    log(f"transpose vec {H}x{W} {dtype}")
    shp = workloads.custom_shape(2, H, W, 3, 16, dtype, H + W, True)
    inp = workloads.make_inputs(shp, "2d")
    u, delta, B, C = (upload_stream(inp, name) for name in ("x", "delta", "B", "C"))
    A, D, bias = (upload_f32(a) for a in (inp.A, inp.D, inp.dt_bias))
    y = torch.empty(u.shape, dtype=torch.float32, device=dev())
    vmb.vmb_mean_scan_fwd(u, delta, A, B, C, D, bias, True, y, layout=vmb.VMB_LAYOUT_2D)
    torch.cuda.synchronize()
    ref, scale = merged_oracle(inp, "mean")
    assert_close(to_f64(y), ref, rtol=FP32_TOL["rtol"], atol=4 * FP32_TOL["atol"], scale=scale,
                 what=f"mean 2d {H}x{W} {dtype}")


# the merge of such planes (bit-exact), by the same tiles
@pytest.mark.parametrize("H,W", [(128, 128), (68, 196), (260, 60), (72, 200), (264, 56)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_merge_vec(H, W, dtype):
    merge_bit_exact((2, 3, H, W), dtype)
