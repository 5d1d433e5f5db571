"""Post-merge norm and gate with a vector of pixels a lane (at least 2048
vectors): images that end inside a vector, channel counts around the groups of
64 up to the most a thread holds (512) and just above, against the fp64 oracle
at the tolerances of the other norm tests."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from gpu_util import BF16_TOL, FP32_TOL, assert_close, dev, log, to_f64, upload_f32
from paper_2412_16602_amd import vmb

pytestmark = pytest.mark.gpu


def draw(shape, rng, dtype):
    a = (rng.standard_normal(shape, dtype=np.float32) + np.float32(0.5)).astype(np.float32)
    if dtype == "bf16":
        a, bits = workloads.bf16_round(a)
        return a, torch.from_numpy(bits.view(np.int16)).to(dev()).view(torch.bfloat16)
    return a, upload_f32(a)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("batch,channels,P,gate,affine", [
    (2050, 1, 8, True, True), (700, 63, 17, True, True), (700, 64, 23, False, True),
    (500, 65, 33, True, False), (300, 192, 65, True, True), (2100, 320, 9, True, True),
    (160, 384, 111, True, True), (90, 385, 196, False, False), (2100, 512, 8, True, True),
    (520, 513, 33, True, True)])
def test_vectors(batch, channels, P, gate, affine, dtype):
    log(f"norm vec b={batch} c={channels} P={P} gate={gate} affine={affine} {dtype}")
    rng = np.random.default_rng(channels + P)
    y, yt = draw((batch, channels, P), rng, dtype)
    z, zt = draw((batch, channels, P), rng, dtype) if gate else (None, None)
    gamma = rng.standard_normal(channels, dtype=np.float32) if affine else None
    beta = rng.standard_normal(channels, dtype=np.float32) if affine else None
    out = torch.empty_like(yt)
    vmb.vmb_ss2d_out_norm(yt, zt, upload_f32(gamma), upload_f32(beta), 1e-5, out)
    torch.cuda.synchronize()
    ref = oracle.out_norm_gate(y, z, gamma, beta, 1e-5)
    assert_close(to_f64(out), ref, **(FP32_TOL if dtype == "f32" else BF16_TOL), what="norm")


# pointers on an element, not on a vector
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_unaligned(dtype):
    log(f"norm vec unaligned {dtype}")
    rng = np.random.default_rng(5)
    shape = (300, 65, 33)

    def shifted(n):
        a, t = draw(shape, rng, dtype)
        s = torch.empty(t.numel() + n, dtype=t.dtype, device=t.device)[n:].view(shape)
        return a, s.copy_(t)

    (y, yt), (z, zt) = shifted(1), shifted(3)
    out = torch.empty(yt.numel() + 1, dtype=yt.dtype, device=yt.device)[1:].view(shape)
    assert yt.data_ptr() % 16 and zt.data_ptr() % 16 and out.data_ptr() % 16
    vmb.vmb_ss2d_out_norm(yt, zt, None, None, 1e-5, out)
    torch.cuda.synchronize()
    ref = oracle.out_norm_gate(y, z, None, None, 1e-5)
    assert_close(to_f64(out), ref, **(FP32_TOL if dtype == "f32" else BF16_TOL), what="norm")
