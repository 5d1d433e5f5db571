"""Full scan with one wave per sequence (every N but 16, N = 16 in bf16 from 1200
rows on and of odd length): run, segment and chunk boundaries, channel-slot tails, the fused
2-D form (planes in LDS, reversed directions whose length is no multiple of a
run), planes beyond LDS, both types and the zero-order-hold option, against the
fp64 oracle at the tolerances of the other scans."""
import dataclasses

import numpy as np
import pytest
import torch

import oracle
import workloads
from gpu_util import BF16_TOL, FP32_TOL, assert_close, dev, log, oracle_seq, run_scan, to_f64
from paper_2412_16602_amd import vmb
from test_gpu_scan import merged_oracle

pytestmark = pytest.mark.gpu


def inputs(b, H, W, c, N, layout, dtype="f32", d_value=0.0):
    shp = workloads.custom_shape(b, H, W, c, N, dtype, 1000 * H + 10 * W + c + N, True)
    return workloads.make_inputs(shp, layout, d_value=d_value)


# runs of 4 (L <= 64) or 8, segments of 16 (L <= 128) and 32 lanes (L <= 256),
# chunks of 512
LENGTHS = [1, 3, 4, 5, 63, 64, 65, 127, 128, 129, 255, 256, 257, 511, 512, 513, 1030]


@pytest.mark.parametrize("N", [1, 4])
@pytest.mark.parametrize("L", LENGTHS)
def test_lengths(L, N):
    log(f"rows full L={L} N={N}")
    inp = inputs(1, 1, L, 5, N, "seq")
    assert_close(to_f64(run_scan(inp, "full", "seq")), oracle_seq(inp, "full", "seq"), **FP32_TOL,
                 what=f"rows L={L} N={N}")


# four waves a workgroup, 4, 2 or 1 channels a wave
@pytest.mark.parametrize("L", [49, 100, 200, 600])
@pytest.mark.parametrize("channels", [1, 2, 7, 16, 17])
@pytest.mark.parametrize("layout", ["seq", "2d"])
def test_channel_slot_tails(layout, channels, L):
    log(f"rows full {layout} L={L} channels={channels}")
    H, W = {49: (7, 7), 100: (10, 10), 200: (8, 25), 600: (20, 30)}[L]
    inp = inputs(2, H, W, channels, 2, layout)
    got = to_f64(run_scan(inp, "full", layout))
    if layout == "seq":
        assert_close(got, oracle_seq(inp, "full", "seq"), **FP32_TOL, what=f"L={L} c={channels}")
    else:
        ref, scale = merged_oracle(inp, "full")
        assert_close(got, ref, rtol=FP32_TOL["rtol"], atol=4 * FP32_TOL["atol"], scale=scale,
                     what=f"2d L={L} c={channels}")


# 80x85 does not fit LDS in fp32 (16 bytes a pixel), 90x93 in neither type (12 in
# bf16) with eight states; with one, both do
MAPS = [(1, 5), (5, 1), (3, 3), (7, 9), (11, 11), (13, 17), (16, 16), (23, 29), (32, 32), (41, 51),
        (80, 85), (90, 93)]


@pytest.mark.parametrize("dtype,out", [("f32", "f32"), ("bf16", "bf16"), ("bf16", "f32")])
@pytest.mark.parametrize("H,W", MAPS)
def test_maps(H, W, dtype, out):
    log(f"rows full 2d {H}x{W} {dtype}->{out}")
    N = 1 if (H + W) % 4 == 0 else 8
    inp = inputs(1, H, W, 3, N, "2d", dtype, d_value=1.0)
    y = run_scan(inp, "full", "2d", out_dtype=torch.bfloat16 if out == "bf16" else torch.float32)
    ref, scale = merged_oracle(inp, "full")
    tol = BF16_TOL if out == "bf16" else FP32_TOL
    assert_close(to_f64(y), ref, rtol=tol["rtol"], atol=4 * tol["atol"], scale=scale,
                 what=f"2d {H}x{W} {dtype}->{out}")


@pytest.mark.parametrize("H,W", [(1, 421), (27, 31), (61, 67), (97, 101)])
@pytest.mark.parametrize("layout", ["seq", "2d"])
def test_odd_bf16_rows_n16(layout, H, W):
    log(f"full {layout} n16 bf16 {H}x{W}")
    inp = inputs(1, H, W, 5, 16, layout, "bf16", d_value=1.0)
    got = to_f64(run_scan(inp, "full", layout, out_dtype=torch.float32))
    if layout == "seq":
        assert_close(got, oracle_seq(inp, "full", "seq"), **FP32_TOL, what=f"odd {H}x{W}")
    else:
        ref, scale = merged_oracle(inp, "full")
        assert_close(got, ref, rtol=FP32_TOL["rtol"], atol=4 * FP32_TOL["atol"], scale=scale,
                     what=f"odd 2d {H}x{W}")


# enough rows for two channels a lane (4096 whole-wave sequences, 8192 and
# 16384 of the segments), with a channel left over, and N = 16 in bf16 (its two
# 2-D cases with one channel a lane)
@pytest.mark.parametrize("layout,b,H,W,c,N,dtype", [
    ("seq", 9, 1, 515, 115, 4, "f32"), ("2d", 9, 17, 31, 115, 1, "bf16"),
    ("2d", 9, 13, 15, 229, 2, "f32"), ("seq", 9, 9, 9, 457, 1, "bf16"),
    ("2d", 9, 7, 7, 459, 8, "f32"), ("2d", 3, 21, 23, 103, 16, "bf16"),
    ("seq", 9, 21, 23, 117, 16, "bf16"), ("2d", 2, 95, 101, 151, 16, "bf16")])
def test_two_channels_a_lane(layout, b, H, W, c, N, dtype):
    log(f"rows {layout} b={b} {H}x{W} c={c} N={N} {dtype}")
    inp = inputs(b, H, W, c, N, layout, dtype, d_value=1.0)
    got = to_f64(run_scan(inp, "full", layout, out_dtype=torch.float32))
    if layout == "seq":
        assert_close(got, oracle_seq(inp, "full", "seq"), **FP32_TOL, what=f"{H}x{W} c={c}")
    else:
        ref, scale = merged_oracle(inp, "full")
        assert_close(got, ref, rtol=FP32_TOL["rtol"], atol=4 * FP32_TOL["atol"], scale=scale,
                     what=f"2d {H}x{W} c={c}")


# N = 16 in bf16: from 1200 rows on in place of the short and chunked kernels
# (1196, 1200), up to 49152 where the tile kernel takes the length (49148, 49152;
# an odd one stays), L = 64 and 65
@pytest.mark.parametrize("b,c,H,W,layout", [
    (13, 23, 6, 12, "seq"), (12, 25, 6, 12, "2d"), (1, 299, 21, 20, "2d"), (1, 300, 21, 20, "seq"),
    (11, 1117, 6, 11, "2d"), (12, 1024, 6, 11, "2d"), (12, 1024, 5, 15, "2d"),
    (12, 1024, 1, 65, "seq"), (5, 61, 8, 8, "2d"), (5, 61, 5, 13, "2d")])
def test_row_limits_n16(layout, b, c, H, W):
    log(f"rows limits {layout} b={b} {H}x{W} c={c}")
    inp = inputs(b, H, W, c, 16, layout, "bf16", d_value=1.0)
    got = to_f64(run_scan(inp, "full", layout, out_dtype=torch.float32))
    if layout == "seq":
        assert_close(got, oracle_seq(inp, "full", "seq"), **FP32_TOL, what=f"{H}x{W} c={c}")
    else:
        ref, scale = merged_oracle(inp, "full")
        assert_close(got, ref, rtol=FP32_TOL["rtol"], atol=4 * FP32_TOL["atol"], scale=scale,
                     what=f"2d {H}x{W} c={c}")


# planes beyond LDS, two channels a lane (one left over): columns gathered from
# the plane (N = 1, 8) or read from its column-major copy (N = 16), sampled channels
@pytest.mark.parametrize("H,W,N,dtype", [(72, 97, 8, "bf16"), (80, 86, 16, "bf16"),
                                         (104, 104, 1, "f32"), (72, 73, 4, "f32")])
def test_large_planes_two_channels(H, W, N, dtype):
    c = 1025
    log(f"rows large planes {H}x{W} c={c} N={N} {dtype}")
    inp = inputs(1, H, W, c, N, "2d", dtype, d_value=1.0)
    got = to_f64(run_scan(inp, "full", "2d", out_dtype=torch.float32))
    ds = [0, 1, 2, 7, 8, 511, 1022, 1023, 1024]
    u = oracle.cross_scan(inp.x)
    seq = oracle.full_scan(u, inp.delta, inp.A, inp.B, inp.C, inp.D, inp.dt_bias, True,
                           sel=[k * c + d for k in range(4) for d in ds])
    seq = np.ascontiguousarray(seq.reshape(1, 4, len(ds), H * W))
    ref, scale = (oracle.cross_merge(a, H, W, "f64") for a in (seq, np.abs(seq)))
    assert_close(got[:, ds], ref, rtol=FP32_TOL["rtol"], atol=4 * FP32_TOL["atol"], scale=scale,
                 what=f"large planes {H}x{W} N={N}")


# the same with one channel a lane, and the vector merge to bf16 (whole vectors)
@pytest.mark.parametrize("H,W,N,dtype", [(104, 108, 1, "f32"), (116, 120, 1, "bf16"),
                                         (100, 132, 8, "bf16"), (100, 132, 16, "bf16")])
def test_large_planes(H, W, N, dtype):
    log(f"rows large planes {H}x{W} N={N} {dtype}")
    inp = inputs(1, H, W, 3, N, "2d", dtype, d_value=1.0)
    got = to_f64(run_scan(inp, "full", "2d"))
    ref, scale = merged_oracle(inp, "full")
    tol = BF16_TOL if dtype == "bf16" else FP32_TOL
    assert_close(got, ref, rtol=tol["rtol"], atol=4 * tol["atol"], scale=scale,
                 what=f"large planes {H}x{W} N={N}")


@pytest.mark.parametrize("N", [1, 8])
@pytest.mark.parametrize("layout,H,W", [("seq", 1, 530), ("2d", 6, 7), ("2d", 23, 25),
                                        ("2d", 90, 91)])
def test_zoh(layout, H, W, N):
    log(f"rows zoh {layout} {H}x{W} N={N}")
    inp = inputs(1, H, W, 6, N, layout)
    got = to_f64(run_scan(inp, "full", layout, options=vmb.VMB_SCAN_ZOH))
    if layout == "seq":
        ref = oracle_seq(inp, "full", "seq", options=oracle.ZOH)
        assert_close(got, ref, **FP32_TOL, what=f"zoh {H}x{W}")
    else:
        ref, scale = merged_oracle(inp, "full", options=oracle.ZOH)
        assert_close(got, ref, rtol=FP32_TOL["rtol"], atol=4 * FP32_TOL["atol"], scale=scale,
                     what=f"zoh 2d {H}x{W}")


def test_no_bias_no_skip_no_softplus():
    log("rows softplus off")
    inp = inputs(1, 15, 19, 6, 2, "2d")
    delta = (np.abs(inp.delta) * 0.05 + 1e-3).astype(np.float32)
    kw = dict(softplus=False, use_bias=False, use_d=False, delta=delta)
    got = to_f64(run_scan(inp, "full", "2d", **kw))
    ref, scale = merged_oracle(inp, "full", **kw)
    assert_close(got, ref, rtol=FP32_TOL["rtol"], atol=4 * FP32_TOL["atol"], scale=scale,
                 what="softplus off")


def with_growth(inp, delta, live):
    """inp with Delta = delta[t] as given (softplus and bias off), A in
    [-1, -0.8] and positive u, B and C, where B is 0 but at the positions that
    ``live`` marks (in each direction's own order)."""
    pos = lambda a: (0.5 + np.abs(a) % 1.0).astype(np.float32)
    N = inp.A.shape[1]
    A = np.broadcast_to(np.linspace(-1.0, -0.8, N, dtype=np.float32), inp.A.shape)
    f = {"delta": np.broadcast_to(delta, inp.delta.shape).astype(np.float32),
         "B": pos(inp.B) * live.astype(np.float32), "C": pos(inp.C)}
    f["x" if inp.u is None else "u"] = pos(inp.x if inp.u is None else inp.u)
    bits = dict(inp.bits or {})
    if inp.shape.dtype == "bf16":
        for name in f:
            f[name], bits[name] = workloads.bf16_round(f[name])
    return dataclasses.replace(inp, A=np.ascontiguousarray(A), bits=bits, **f)


def check_growth(inp, layout, rtol, options=0):
    kw = dict(softplus=False, use_bias=False, use_d=False)
    got = to_f64(run_scan(inp, "full", layout, out_dtype=torch.float32, **kw,
                          options=vmb.VMB_SCAN_ZOH if options else None))
    if layout == "seq":
        ref, scale = oracle_seq(inp, "full", "seq", options=options, **kw), None
    else:
        ref, scale = merged_oracle(inp, "full", options=options, **kw)
    assert_close(got, ref, rtol=rtol, atol=1e-5, scale=scale, what="growing states")


# Factors above 1 whose product over the sequence (or a chunk of it) is beyond
# fp32, on a state that is 0 until the last positions: finite, step by step.
# Each step rounds by at most 3 * 2^-24 (exponent, exp2, fma), 160 of them at most.
@pytest.mark.parametrize("layout,b,H,W,c,N,dtype,step", [
    ("seq", 1, 1, 49, 7, 1, "f32", 3.0), ("seq", 1, 1, 120, 9, 2, "bf16", 1.5),
    ("seq", 1, 1, 250, 5, 4, "f32", 1.0), ("seq", 1, 1, 1030, 5, 4, "f32", 0.25),
    ("seq", 1, 1, 700, 300, 16, "bf16", 0.25), ("seq", 1, 1, 701, 3, 16, "bf16", 0.25),
    ("2d", 1, 27, 31, 3, 16, "bf16", 0.25), ("2d", 1, 7, 9, 5, 2, "f32", 3.0),
    ("2d", 1, 23, 29, 3, 8, "f32", 0.25), ("2d", 1, 90, 93, 2, 8, "bf16", 0.25)])
def test_growing_states(layout, b, H, W, c, N, dtype, step):
    log(f"rows growing {layout} {H}x{W} N={N} {dtype}")
    inp = inputs(b, H, W, c, N, layout, dtype)
    L = H * W
    live = np.arange(L) >= L - int(40 / step)
    inp = with_growth(inp, np.full(L, -step, np.float32), live)
    # (zero-order hold with N = 16: other kernels for even lengths)
    for options in (0, oracle.ZOH) if N < 16 or L % 2 else (0,):
        check_growth(inp, layout, 160 * 3 * 2.0 ** -24, options)


# a state that decays to 1e-28 before a chunk whose product of factors is 1e55
def test_growing_small_state():
    log("rows growing small state")
    inp = inputs(1, 1, 1030, 5, 1, "seq")
    delta = np.zeros(1030, np.float32)
    delta[455:460], delta[460:510], delta[520:571] = 1.0, 1.3, -2.5
    check_growth(with_growth(inp, delta, np.arange(1030) < 460), "seq", 110 * 3 * 2.0 ** -24 + 1e-5)


# A = -inf forgets the state at every position; a plane whose length is no
# multiple of a run has identity positions ahead of its reversed directions
@pytest.mark.parametrize("layout,H,W", [("2d", 7, 9), ("2d", 11, 11), ("2d", 23, 29),
                                        ("seq", 1, 513)])
def test_infinite_decay(layout, H, W):
    log(f"rows A = -inf {layout} {H}x{W}")
    inp = inputs(1, H, W, 5, 2, layout)
    inp.A[:, 0] = -np.inf
    got = to_f64(run_scan(inp, "full", layout))
    if layout == "seq":
        ref, scale = oracle_seq(inp, "full", layout), None
    else:
        ref, scale = merged_oracle(inp, "full")
    assert_close(got, ref, rtol=FP32_TOL["rtol"], atol=4 * FP32_TOL["atol"], scale=scale,
                 what="A = -inf")


# an infinite input: before it, and in the other channels, nothing changes
@pytest.mark.parametrize("L", [49, 200, 1030])
def test_infinite_input(L):
    log(f"rows u = inf L={L}")
    inp = inputs(1, 1, L, 6, 2, "seq")
    at = L * 2 // 3
    inp.u[0, 1, 3, at] = np.inf
    got, ref = to_f64(run_scan(inp, "full", "seq")), oracle_seq(inp, "full", "seq")
    bad = ~np.isfinite(ref)
    assert bad[0, 1, 3, at:].all() and bad.sum() == L - at
    assert not np.isfinite(got[bad]).any()
    assert_close(np.where(bad, 0.0, got), np.where(bad, 0.0, ref), **FP32_TOL, what="u = inf")


# more channels than one launch takes (2^28 with one wave for 16, 2^26 with one
# workgroup for 4): the outputs repeat those of a few channels, bit for bit
@pytest.mark.parametrize("layout,channels", [("seq", 2 ** 28 + 5), ("2d", 2 ** 26 + 3)])
def test_many_channels(layout, channels):
    log(f"rows {layout} channels={channels}")
    two_d, K, few = layout == "2d", 4 if layout == "2d" else 1, 997
    g = torch.Generator().manual_seed(1)
    period = lambda n: torch.rand(n, generator=g).add_(0.5).to(torch.bfloat16).to(dev())
    u1, d1 = period(few), period(few)
    B = torch.ones((1, K, 1, 1), dtype=torch.bfloat16, device=dev())

    def call(c):
        rep = lambda p: p.repeat(-(-c // few))[:c]
        u = rep(u1).view(1, 1, c, 1)
        delta = rep(d1).view(1, 1, c, 1).expand(1, K, c, 1).contiguous()
        A = torch.full((K * c, 1), -1.0, device=dev())
        y = torch.empty_like(u)
        lay = vmb.VMB_LAYOUT_2D if two_d else vmb.VMB_LAYOUT_SEQ
        if two_d:
            u, y = u.view(1, c, 1, 1), y.view(1, c, 1, 1)
        vmb.vmb_selective_scan_fwd_ex(u, delta, A, B, B, None, None, False, y, vmb.VMB_SCAN_ZOH,
                                      layout=lay)
        return y.view(-1)

    want = call(few).repeat(-(-channels // few))[:channels]
    assert torch.isfinite(want[:few].float()).all()
    assert torch.equal(call(channels), want)
