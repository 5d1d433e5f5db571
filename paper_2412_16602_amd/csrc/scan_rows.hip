// scan_rows.hip -- full selective scan, one wave per sequence (any N; the
// path of every N but 16, of N = 16 in bf16 between 1200 and 49152 rows, and of
// the N = 16 forms the other kernels refuse: bf16 rows of odd length).
//
// Same recurrence as scan_full.hip (Appendix A: eq. 3, eq. 4 first line,
// eq. 6). Lanes own runs of T = 8 (or 4) consecutive positions; a wave walks
// its sequence in chunks of 64 T positions, sequences of up to 32 T (16 T)
// positions share a wave, 2 (4) channels of a direction each in a segment of
// 32 (16) lanes. Per state a lane forms a_i = exp(Delta_i A_n) and
// b_i = Delta_i B_i u_i for its run and folds them into the run's aggregate,
// an inclusive DPP scan over the wave (segment) joins the runs, and the lane
// re-walks its run from the state entering it, accumulating y_i += C_i h_i.
// The state leaving a chunk is kept per state in lane n of one register.
//
// What bounds it: instruction issue (32 x 56x56, 192 channels, bf16, sequence
// layout: 250 cycles a SIMD per 64 positions at N = 1, of which softplus is
// about 45, and 46 more per state), near the rate of a copy in fp32 (4.1 TB/s).
// delta, B and C are read as whole 16-byte vectors of a run, the next state's
// B and C (and the next chunk's delta) in flight while the current ones are in
// use: their values are unpacked before those loads are issued (pin), or the
// loop would wait for them at the end of the step that issued them.
// At the same shape, 2-D, N = 1: one lane per channel 1830 us; this kernel 106
// (176 with an output plane per direction, two workgroups a CU instead of
// four, and the early wait). With few sequences latency: 2 x 97x101, 200
// channels, N = 16 in bf16 are 1600 waves on 1024 SIMDs, 168 us, of which a wave
// lives 0.86 on average and issues a VALU instruction every 10.5 cycles.
//
// 2-D layout, planes that fit LDS (kFused): a workgroup owns a channel (2 or
// 4 short ones) with one wave per direction. The input plane is copied into
// LDS in both scan orders, and each order has one output plane, which its
// forward and its reversed direction share (see step 4); at the end the two
// are summed and stored, in the association of the cross-merge,
// (y0 + y2) + (y1 + y3). Per-direction outputs never reach memory (the merge
// pass it replaces moved 32 bytes per pixel and channel). All LDS runs are
// aligned vectors: the reversed directions start their runs at the padded end
// of the plane, with identity positions (Delta = 0, B = 0) ahead of the first
// pixel.
//
// Values that are not finite: see walk_positions.
#include "vmb_internal.h"

namespace vmb {
namespace {

constexpr int kWave = 64;
constexpr int kRowWaves = 4;
constexpr int kRowThreads = kRowWaves * kWave;
constexpr int kWaveShr1 = 0x138;  // DPP wave_shr:1 (GFX9 encoding)

enum RowMode { kSeq = 0, kFused = 1, kMapRows = 2 };

__device__ __forceinline__ float shr1(float old, float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, old),
                                                                 __builtin_bit_cast(int, v),
                                                                 kWaveShr1, 0xf, 0xf, false));
}
__device__ __forceinline__ float lane_value(float v, int lane) {
    return __builtin_bit_cast(float,
                              __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane));
}

// T elements as they lie in memory.
template <typename Tin, int T>
struct Run {
    static constexpr int kWords = T * static_cast<int>(sizeof(Tin)) / 4;
    uint32_t w[kWords];
};
template <int T>
__device__ __forceinline__ float run_at(const Run<float, T>& r, int i) {
    return __uint_as_float(r.w[i]);
}
template <int T>
__device__ __forceinline__ float run_at(const Run<bf16_t, T>& r, int i) {
    return __uint_as_float((i & 1) ? r.w[i / 2] & 0xffff0000u : r.w[i / 2] << 16);
}

// The run at element offset off from base: one vector when its T elements lie
// inside the tensor, that is lo <= off and off + T <= hi (they may belong to
// the next or previous row: positions outside the sequence are never used).
// At the ends of the tensor the row's own elements [first, last] are read one
// by one (a rolled loop that shifts them in from the top, to stay small).
template <int T>
__device__ __forceinline__ void shift_in(Run<float, T>& r, float e) {
#pragma unroll
    for (int i = T - 1; i > 0; --i) r.w[i] = r.w[i - 1];
    r.w[0] = __float_as_uint(e);
}
template <int T>
__device__ __forceinline__ void shift_in(Run<bf16_t, T>& r, bf16_t e) {
#pragma unroll
    for (int i = Run<bf16_t, T>::kWords - 1; i > 0; --i)
        r.w[i] = (r.w[i] << 16) | (r.w[i - 1] >> 16);
    r.w[0] = (r.w[0] << 16) | e.bits;
}
template <typename Tin, int T>
__device__ __forceinline__ void load_run(const Tin* base, int off, int lo, int hi, int first,
                                         int last, Run<Tin, T>& r) {
    if (off >= lo && off + T <= hi) {
        __builtin_memcpy(&r, base + off, sizeof(r));
    } else {
#pragma unroll
        for (int i = 0; i < Run<Tin, T>::kWords; ++i) r.w[i] = 0;
        if (off <= last) {
#pragma unroll 1
            for (int i = T - 1; i >= 0; --i) {
                const int o = off + i < first ? first : (off + i > last ? last : off + i);
                shift_in<T>(r, base[o]);
            }
        }
    }
}

// LDS planes: T fp32 values, aligned, forwards or reversed.
template <int T>
__device__ __forceinline__ void put_run(float* p, const float (&v)[T], bool rev, bool add) {
    float4 f[T / 4];
#pragma unroll
    for (int q = 0; q < T / 4; ++q)
        f[q] = rev ? make_float4(v[T - 1 - 4 * q], v[T - 2 - 4 * q], v[T - 3 - 4 * q],
                                 v[T - 4 - 4 * q])
                   : make_float4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
    if (add) {
#pragma unroll
        for (int q = 0; q < T / 4; ++q) {
            const float4 o = *reinterpret_cast<const float4*>(p + 4 * q);
            f[q].x += o.x;
            f[q].y += o.y;
            f[q].z += o.z;
            f[q].w += o.w;
        }
    }
#pragma unroll
    for (int q = 0; q < T / 4; ++q) *reinterpret_cast<float4*>(p + 4 * q) = f[q];
}

template <int S>
__device__ __forceinline__ void scan_lanes(float& P, float& H) {
    if constexpr (S == kWave)
        wave_scan(P, H);
    else
        seg_scan<S>(P, H);
}

// distance (>= 0) to the end of a tensor or of a row, kept in 32 bits
__device__ __forceinline__ int near(int64_t v) {
    return (static_cast<uint64_t>(v) >> 30) ? (1 << 30) : static_cast<int>(v);
}

// values formed here and not sunk past the loads that follow
template <int T>
__device__ __forceinline__ void pin(float (&v)[T]) {
#pragma unroll
    for (int i = 0; i < T; ++i) asm volatile("" : "+v"(v[i]));
}

// smallest number of waves per SIMD the registers are budgeted for: what the
// fused form's LDS admits at 56x56 (12 or 16 bytes a pixel and channel), and
// the same budget elsewhere (two fp32 chains at a time need about 150
// registers)
template <typename Tin, int kChains, int kMode>
constexpr int row_waves() {
    return kChains == 2 && (sizeof(Tin) == 4 || kMode == kMapRows) ? 3 : 4;
}

struct RowArgs {
    const void* u;
    const void* delta;
    const float* A;
    const void* B;
    const void* C;
    const float* D;
    const float* dt_bias;
    void* y;
    const void* xt;
    int batch, K, Dc, N, H, W, softplus;
    int64_t L;
    int groups;     // workgroups per (batch, direction), or per batch when fused
    int first;      // the first of them (in a launch over part of the channels)
    unsigned n_wg;  // whole grid, 0 when it is not renumbered
};

// Where a wave works: batch entry, direction, first channel, number of channels.
struct Place {
    int b, k, d0, nc;
};
// Workgroup i runs on XCD i % 8 (own L2): each XCD takes a contiguous
// range, so the channels that share B and C rows share an L2.
template <int kMode, int kPlanes>
__device__ __forceinline__ Place place_of(const RowArgs& g, int wv) {
    int grp;
    Place p;
    if (g.n_wg) {
        const unsigned bid = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
        const unsigned per = g.n_wg / 8, rem = g.n_wg % 8, xcd = bid % 8, slot = bid / 8;
        unsigned id = xcd * per + (xcd < rem ? xcd : rem) + slot;
        grp = static_cast<int>(id % static_cast<unsigned>(g.groups));
        id /= static_cast<unsigned>(g.groups);
        p.k = static_cast<int>(id % gridDim.y);
        p.b = static_cast<int>(id / gridDim.y);
    } else {
        grp = blockIdx.x;
        p.k = blockIdx.y;
        p.b = blockIdx.z;
    }
    grp += g.first;
    if constexpr (kMode == kFused) p.k = wv;  // gridDim.y is 1
    p.d0 = kMode == kFused ? grp * kPlanes : (grp * kRowWaves + wv) * kPlanes;
    p.nc = g.Dc - p.d0 < kPlanes ? g.Dc - p.d0 : kPlanes;
    return p;
}

// LDS of the fused form: planes (rows of row_len elements) of the input in both
// scan orders, then of the outputs of both.
__host__ __device__ inline int row_len(int64_t L, int T) {
    return static_cast<int>((L + T - 1) / T * T);
}

// Fused form: the sums of the two scan orders, stored to y, four pixels a
// thread at a time. Returns 0, or NaN where a sum was not finite.
template <int T, int kPlanes, typename Tin, typename Tout>
__device__ __forceinline__ float fold_planes(const RowArgs& g, const Place& place, char* lds) {
    constexpr int kThr = kRowThreads / kPlanes;  // threads per plane
    const int ch = threadIdx.x / kThr;
    if (ch >= place.nc) return 0.0f;
    const int H = g.H, W = g.W, L = static_cast<int>(g.L), Lp = row_len(L, T);
    Tout* out =
        static_cast<Tout*>(g.y) + (static_cast<size_t>(place.b) * g.Dc + place.d0 + ch) * L;
    const float* y_planes = reinterpret_cast<const float*>(lds + 2 * kPlanes * Lp * sizeof(Tin));
    const float* yr = y_planes + ch * Lp;
    const float* yc = y_planes + (kPlanes + ch) * Lp;
    int p = (threadIdx.x % kThr) * 4;
    int h = p / W, w = p - h * W;
    const int dh = 4 * kThr / W, dw = 4 * kThr - dh * W;
    float bad = 0.0f;
    for (; p < L; p += 4 * kThr) {
        const float4 r = *reinterpret_cast<const float4*>(yr + p);  // whole runs: Lp % 4 == 0
        const float rv[4] = {r.x, r.y, r.z, r.w};
        float sum[4];
        Tout o[4];
        int hh = h, ww = w;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            sum[i] = rv[i] + yc[p + i < L ? ww * H + hh : 0];
            o[i] = from_f32<Tout>(sum[i]);
            if (++ww == W) { ww = 0; ++hh; }
        }
        if (p + 4 <= L) {
            __builtin_memcpy(out + p, o, sizeof(o));
#pragma unroll
            for (int i = 0; i < 4; ++i) bad = __builtin_fmaf(sum[i], 0.0f, bad);
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (p + i < L) {
                    out[p + i] = o[i];
                    bad = __builtin_fmaf(sum[i], 0.0f, bad);
                }
        }
        w += dw;
        h += dh;
        if (w >= W) { w -= W; ++h; }
    }
    return bad;
}

// The kernel's arguments, read once more: for a path that is hardly ever taken
// and shall hold no registers in the one that always is.
__device__ __forceinline__ RowArgs args_again() {
    typedef const __attribute__((address_space(4))) RowArgs* Args;
    Args args = (Args)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(args));
    return *(const RowArgs*)args;
}

// The wave's sequences once more, position after position: lane 16 j + n has
// state n of the j-th of four channels at a time. For outputs that came out
// infinite or NaN: a product of factors above 1 over several runs may leave the
// range of fp32 (0.2 a position over 512 is enough) where the states
// themselves, zero or small, do not; the identity positions ahead of a reversed
// plane form 0 A, NaN for an infinite A; and values that are not finite by
// themselves are to be what the recurrence makes of them. (A state that is not
// finite makes every output that it enters so, whatever C is.) About as slow as
// a lane per channel, and never reached by states that decay.
template <int T, int kPlanes, typename Tin, typename Tout, int kMode, bool kZoh>
__device__ __forceinline__ void walk_positions(int wv, char* lds) {
    const RowArgs g = args_again();
    const Place p = place_of<kMode, kPlanes>(g, wv);
    const int lane = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    const int n = lane % 16, N = g.N;
    const int64_t L = g.L, bk = static_cast<int64_t>(p.b) * g.K + p.k;
    const Tin* Bn = static_cast<const Tin*>(g.B) + (bk * N + (n < N ? n : 0)) * L;
    const Tin* Cn = static_cast<const Tin*>(g.C) + (bk * N + (n < N ? n : 0)) * L;
    const bool rev = p.k >= 2;
    const int Lp = kMode == kFused ? row_len(L, T) : 0;
    float* planes = reinterpret_cast<float*>(lds + 2 * kPlanes * Lp * sizeof(Tin)) +
                    (p.k & 1) * kPlanes * Lp;
#pragma unroll 1
    for (int j0 = 0; j0 < p.nc; j0 += kWave / 16) {
        const int ch = j0 + lane / 16;
        const int d = p.d0 + (ch < p.nc ? ch : p.nc - 1), c = p.k * g.Dc + d;
        const int64_t row = (bk * g.Dc + d) * L;
        const Tin* drow = static_cast<const Tin*>(g.delta) + row;
        const Tin* urow = static_cast<const Tin*>(g.u) +
                          (kMode == kSeq ? row : (static_cast<int64_t>(p.b) * g.Dc + d) * L);
        const float an = n < N ? g.A[static_cast<size_t>(c) * N + n] : 0.0f;
        const float inv_a = kZoh ? 1.0f / an : 0.0f;
        const float bias = g.dt_bias ? g.dt_bias[c] : 0.0f, dskip = g.D ? g.D[c] : 0.0f;
        float h = 0.0f;
#pragma unroll 1
        for (int64_t t = 0; t < L; ++t) {
            const float ut = to_f32(
                urow[kMode == kSeq ? t : pixel_of(p.k, static_cast<int>(t), g.H, g.W)]);
            const float dl = timescale(to_f32(drow[t]) + bias, g.softplus != 0);
            const float x2 = dl * kLog2e * an, a = fast_exp2(x2), du = dl * ut;
            const float q = kZoh ? zoh_q(x2, a, du, ut, inv_a) : du;
            h = __builtin_fmaf(a, h, q * to_f32(Bn[t]));
            float y = n < N ? to_f32(Cn[t]) * h : 0.0f;
#pragma unroll
            for (int m = 1; m < 16; m *= 2) y += __shfl_xor(y, m, kWave);
            if (n != 0 || ch >= p.nc) continue;
            y = __builtin_fmaf(dskip, ut, y);
            if constexpr (kMode == kFused) {
                // the reversed direction adds to its plane
                float* o = planes + ch * Lp + (rev ? L - 1 - t : t);
                *o = rev ? *o + y : y;
            } else {
                static_cast<Tout*>(g.y)[row + t] = from_f32<Tout>(y);
            }
        }
    }
}

template <int S, int T, int CH, int NP, typename Tin, typename Tout, int kMode, bool kZoh, bool kN1>
__global__ __launch_bounds__(kRowThreads, (row_waves<Tin, CH * NP, kMode>())) void k_full_scan_rows(
    const RowArgs g) {
    constexpr int kCpw = kWave / S;   // sequences (channels) side by side in a wave
    constexpr int kPlanes = CH * kCpw;  // channels of a wave
    constexpr int kX = CH * NP;       // recurrences a lane runs at a time: x = h NP + s
    constexpr int kChunk = S * T;
    extern __shared__ __align__(16) char lds[];

    const int tid = threadIdx.x;
    const int lane = tid % kWave;
    const int wv = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int cw = lane / S, sl = lane % S;
    const int Dc = g.Dc, N = kN1 ? 1 : g.N;  // a multiple of NP
    const int64_t L = g.L;

    const Place here = place_of<kMode, kPlanes>(g, wv);
    const int b = here.b, k = here.k, d0 = here.d0;
    if (kMode != kFused && d0 >= Dc) return;
    const int nc = here.nc;
    int slot_of[CH], cc[CH];  // this lane's channels; slots past nc repeat the last, unstored
#pragma unroll
    for (int h = 0; h < CH; ++h) {
        slot_of[h] = h * kCpw + cw;
        cc[h] = slot_of[h] < nc ? slot_of[h] : nc - 1;
    }
    const int64_t bk = static_cast<int64_t>(b) * g.K + k;
    const int iL = kMode == kSeq ? 0 : static_cast<int>(L);  // 2-D maps: L = H * W fits an int

    // fused: LDS planes (rows of Lp elements): input in both scan orders,
    // then the outputs of both
    const int Lp = kMode == kFused ? row_len(iL, T) : 0;
    Tin* u_rows = reinterpret_cast<Tin*>(lds);
    Tin* u_cols = u_rows + kPlanes * Lp;
    float* y_planes = reinterpret_cast<float*>(u_cols + kPlanes * Lp);
    const bool rev = kMode == kFused && k >= 2;
    const int lead = rev ? Lp - iL : 0;  // identity positions ahead of the sequence

    const int64_t rows = static_cast<int64_t>(g.batch) * g.K;
    const Tin* delta = static_cast<const Tin*>(g.delta);
    const Tin* Bm = static_cast<const Tin*>(g.B);
    const Tin* Cm = static_cast<const Tin*>(g.C);
    const bool sp = g.softplus != 0;
    float bias[CH], dskip[CH];
    const float* Ac[CH];
    int64_t row0[CH];  // delta row of the channel (of the first of its segments)
    int loff[CH];      // this lane's first position from there
#pragma unroll
    for (int h = 0; h < CH; ++h) {
        const int c = k * Dc + d0 + cc[h];
        bias[h] = g.dt_bias ? g.dt_bias[c] : 0.0f;
        dskip[h] = g.D ? g.D[c] : 0.0f;
        Ac[h] = g.A + static_cast<size_t>(c) * N;
        // one channel a wave: cc is uniform and the base takes it
        row0[h] = (bk * Dc + d0 + (kCpw > 1 ? 0 : (h < nc ? h : nc - 1))) * L;
        loff[h] = (kCpw > 1 ? cc[h] * static_cast<int>(L) : 0) + sl * T - lead;
    }

    // one chunk's run of a row: base at the chunk, lane offsets in 32 bits
    auto load_row = [&](const Tin* base, int64_t c0, int h, Run<Tin, T>& r) {
        const int row_first = kCpw > 1 ? cc[h] * static_cast<int>(L) : -near(c0);
        const int row_last = kCpw > 1 ? row_first + static_cast<int>(L) - 1 : near(L - 1 - c0);
        load_run<Tin, T>(base + row0[h] + c0, loff[h], -near(row0[h] + c0),
                         near(rows * Dc * L - row0[h] - c0), row_first, row_last, r);
    };
    auto load_state = [&](const Tin* base, int64_t c0, int n, Run<Tin, T>& r) {
        const int64_t at = (bk * N + n) * L + c0;
        load_run<Tin, T>(base + at, sl * T - lead, -near(at), near(rows * N * L - at), -near(c0),
                         near(L - 1 - c0), r);
    };
    // u of a chunk from global memory: the sequence's own row, or (kMapRows)
    // the plane read in direction k's order
    auto load_u = [&](int64_t c0, int h, Run<Tin, T>& r, bool& reversed) {
        reversed = false;
        const Tin* u = static_cast<const Tin*>(g.u);
        if constexpr (kMode == kSeq) {
            load_row(u, c0, h, r);
        } else {
            const Tin* src = (k & 1) && g.xt ? static_cast<const Tin*>(g.xt) : u;
            const int64_t p0 = (static_cast<int64_t>(b) * Dc + d0 + (h < nc ? h : nc - 1)) * L;
            const int64_t t0 = c0 + sl * T;
            if (!(k & 1) || g.xt) {
                reversed = k >= 2;
                const int64_t at = p0 + (reversed ? L - c0 : c0);
                load_run<Tin, T>(src + at, reversed ? -T - sl * T : sl * T, -near(at),
                                 near(static_cast<int64_t>(g.batch) * Dc * L - at),
                                 reversed ? -near(L - c0) : -near(c0),
                                 reversed ? near(c0) - 1 : near(L - 1 - c0), r);
            } else {
                // column-major gather; positions past the end read the last pixel
                Tin e[T];
                const int ts = t0 < L ? static_cast<int>(t0) : iL - 1;
                const int tt = k >= 2 ? iL - 1 - ts : ts;
                int pw = tt / g.H, ph = tt - pw * g.H;
#pragma unroll
                for (int i = 0; i < T; ++i) {
                    e[i] = src[p0 + static_cast<int64_t>(ph) * g.W + pw];
                    if (t0 + i + 1 < L) {
                        if (k < 2) {
                            if (++ph == g.H) { ph = 0; ++pw; }
                        } else {
                            if (--ph < 0) { ph = g.H - 1; --pw; }
                        }
                    }
                }
                __builtin_memcpy(&r, e, sizeof(r));
            }
        }
    };

    Run<Tin, T> draw[CH], uraw[CH];
    bool urev = false;
    auto load_chunk = [&](int64_t c0) {
#pragma unroll
        for (int h = 0; h < CH; ++h) {
            load_row(delta, c0, h, draw[h]);
            if constexpr (kMode != kFused) load_u(c0, h, uraw[h], urev);
        }
    };
    load_chunk(0);

    Run<Tin, T> braw[NP], craw[NP];
    float araw[kX];
    auto load_states = [&](int64_t c0, int n) {
#pragma unroll
        for (int s = 0; s < NP; ++s) {
            load_state(Bm, c0, n + s, braw[s]);
            load_state(Cm, c0, n + s, craw[s]);
#pragma unroll
            for (int h = 0; h < CH; ++h) araw[h * NP + s] = Ac[h][n + s];
        }
    };
    load_states(0, 0);

    if constexpr (kMode == kFused) {
        // the channels' planes into both scan orders, vectors of kPer pixels
        constexpr int kPer = 16 / static_cast<int>(sizeof(Tin));
        constexpr int kThr = kRowThreads / kPlanes;  // threads per plane
        const int ch = tid / kThr;
        const Tin* x = static_cast<const Tin*>(g.u) +
                       (static_cast<size_t>(b) * Dc + d0 + (ch < nc ? ch : 0)) * iL;
        Tin* pr = u_rows + ch * Lp;
        Tin* pc = u_cols + ch * Lp;
        for (int p = (tid % kThr) * kPer; p < iL; p += kThr * kPer) {
            Tin v[kPer];
            const int n = iL - p < kPer ? iL - p : kPer;
            int h = p / g.W, w = p - h * g.W;
            if (n == kPer) {
                __builtin_memcpy(v, x + p, 16);
                __builtin_memcpy(__builtin_assume_aligned(pr + p, T == 4 ? 8 : 16), v, 16);
#pragma unroll
                for (int i = 0; i < kPer; ++i) {
                    pc[w * g.H + h] = v[i];
                    if (++w == g.W) { w = 0; ++h; }
                }
            } else {
#pragma unroll 1
                for (int i = 0; i < n; ++i) {
                    const Tin e = x[p + i];
                    pr[p + i] = e;
                    pc[w * g.H + h] = e;
                    if (++w == g.W) { w = 0; ++h; }
                }
            }
        }
        __syncthreads();
    }
    // the middle chunk, around which the two directions of a plane exchange
    // (kFused, step 4)
    const int chunks = kMode == kFused ? (Lp + kChunk - 1) / kChunk : 0;
    const int64_t middle = kMode == kFused ? static_cast<int64_t>((chunks - 1) / 2) * kChunk : -1;

    float carry[CH];  // lane n: state n leaving the previous chunk
#pragma unroll
    for (int h = 0; h < CH; ++h) carry[h] = 0.0f;
    int bad = 0;  // outputs that are not finite came up (kFused: see fold_planes)
    for (int64_t c0 = 0; c0 < L + lead; c0 += kChunk) {
        // 1. per-position products of the runs
        int at = 0;  // fused: the run's first element in its plane
        bool in_plane = true;
        if constexpr (kMode == kFused) {
            const int t0 = static_cast<int>(c0) + sl * T;
            at = rev ? Lp - T - t0 : t0;
            in_plane = at >= 0 && at < Lp;
        }
        const bool led = kMode == kFused && lead > 0 && c0 == 0;
        float uv[CH][T], dl2[CH][T], du[CH][T], yv[CH][T], s2[CH];
#pragma unroll
        for (int h = 0; h < CH; ++h) {
            if constexpr (kMode == kFused) {
                const Tin* src = ((k & 1) ? u_cols : u_rows) + cc[h] * Lp + (in_plane ? at : 0);
                Run<Tin, T> r;
                __builtin_memcpy(&r, __builtin_assume_aligned(src, sizeof(Tin) * T < 16 ? 8 : 16),
                                 sizeof(r));
#pragma unroll
                for (int i = 0; i < T; ++i) uv[h][i] = rev ? run_at(r, T - 1 - i) : run_at(r, i);
            } else {
#pragma unroll
                for (int i = 0; i < T; ++i)
                    uv[h][i] = urev ? run_at(uraw[h], T - 1 - i) : run_at(uraw[h], i);
            }
#pragma unroll
            for (int i = 0; i < T; ++i) dl2[h][i] = run_at(draw[h], i) + bias[h];
            if (sp) {
#pragma unroll
                for (int i = 0; i < T; ++i) dl2[h][i] = softplus(dl2[h][i]);
            }
            if (led) {  // identity positions ahead of a reversed sequence
#pragma unroll
                for (int i = 0; i < T; ++i) {
                    if (sl == 0 && i < lead) dl2[h][i] = uv[h][i] = 0.0f;
                    asm volatile("" : "+v"(dl2[h][i]), "+v"(uv[h][i]));  // a branch of its own
                }
            }
            s2[h] = 0.0f;
#pragma unroll
            for (int i = 0; i < T; ++i) {
                du[h][i] = dl2[h][i] * uv[h][i];
                dl2[h][i] *= kLog2e;
                yv[h][i] = dskip[h] * uv[h][i];
                s2[h] += dl2[h][i];
            }
            // the loads below reuse the raw registers
            pin(dl2[h]), pin(du[h]), pin(yv[h]);
        }
        // 2. the next chunk's delta (and u) in flight during the states
        const bool more = c0 + kChunk < L + lead;
        if (more) load_chunk(c0 + kChunk);
        // 3. the states, NP at a time, for each of the lane's channels: the
        //    recurrences' chains are independent of each other
#pragma unroll 1
        for (int n = 0; n < N; n += NP) {
            float an[kX], a[kX][T], bu[kX][T], bv[NP][T], cv[NP][T], P[kX], Hs[kX];
#pragma unroll
            for (int s = 0; s < NP; ++s) {
#pragma unroll
                for (int i = 0; i < T; ++i) {
                    bv[s][i] = run_at(braw[s], i);
                    cv[s][i] = run_at(craw[s], i);
                }
                // the loads below reuse the raw registers
                pin(bv[s]), pin(cv[s]);
                if (led) {
#pragma unroll
                    for (int i = 0; i < T; ++i) {
                        if (sl == 0 && i < lead) bv[s][i] = 0.0f;
                        asm volatile("" : "+v"(bv[s][i]));
                    }
                }
            }
#pragma unroll
            for (int x = 0; x < kX; ++x) {
                an[x] = araw[x];
                asm volatile("" : "+v"(an[x]));
            }
            if (n + NP < N)
                load_states(c0, n + NP);
            else if (more)
                load_states(c0 + kChunk, 0);
#pragma unroll
            for (int x = 0; x < kX; ++x) {
                const int h = x / NP, s = x % NP;
                const float inv_a = kZoh ? 1.0f / an[x] : 0.0f;
                float agg = 0.0f;
#pragma unroll
                for (int i = 0; i < T; ++i) {
                    const float x2 = dl2[h][i] * an[x];
                    a[x][i] = fast_exp2(x2);
                    const float q = kZoh ? zoh_q(x2, a[x][i], du[h][i], uv[h][i], inv_a) : du[h][i];
                    bu[x][i] = q * bv[s][i];
                    agg = i == 0 ? bu[x][0] : __builtin_fmaf(a[x][i], agg, bu[x][i]);
                }
                P[x] = fast_exp2(s2[h] * an[x]);
                Hs[x] = agg;
            }
            if constexpr (kX == 2 && S == kWave) {
                wave_scan2(P[0], Hs[0], P[1], Hs[1]);
            } else {
#pragma unroll
                for (int x = 0; x < kX; ++x) scan_lanes<S>(P[x], Hs[x]);
            }
#pragma unroll
            for (int x = 0; x < kX; ++x) {
                const int h = x / NP, s = x % NP;
                float hs;
                if constexpr (S == kWave) {
                    const float cin = lane_value(carry[h], n + s);
                    const float out = __builtin_fmaf(P[x], cin, Hs[x]);
                    hs = shr1(cin, out);  // lane 0 keeps the chunk's carry
                    carry[h] = lane == n + s ? lane_value(out, kWave - 1) : carry[h];
                } else {
                    const float in = shr1(0.0f, Hs[x]);
                    hs = sl == 0 ? 0.0f : in;
                }
#pragma unroll
                for (int i = 0; i < T; ++i) {
                    hs = __builtin_fmaf(a[x][i], hs, bu[x][i]);
                    yv[h][i] = __builtin_fmaf(cv[s][i], hs, yv[h][i]);
                }
            }
        }
        if constexpr (kMode != kFused) {
            bool any = false;
#pragma unroll
            for (int h = 0; h < CH; ++h) any |= !__builtin_isfinite(yv[h][0]);
            if (__builtin_amdgcn_ballot_w64(any) != 0) bad = 1;
        }
        // 4. outputs
        if constexpr (kMode == kFused) {
            // A plane takes the forward and the reversed direction of its
            // scan order: whichever reaches a run first (in chunks; the
            // forward one on a tie) stores it, the other adds to it, so the
            // sum is the same whatever the waves' timing. Runs reached in
            // different chunks are reached on different sides of the middle
            // one, so only that chunk needs barriers: before it, between the
            // forward and the reversed waves, and after it.
            const int other = (rev ? at : Lp - T - at) / kChunk;
            const int mine = static_cast<int>(c0 / kChunk);
            const bool add = in_plane && (rev ? other <= mine : other < mine);
            float* dst = y_planes + ((k & 1) * kPlanes + cw) * Lp + at;
            auto put = [&]() {
                if (in_plane)
#pragma unroll
                    for (int h = 0; h < CH; ++h) put_run<T>(dst + h * kCpw * Lp, yv[h], rev, add);
            };
            if (c0 == middle) __syncthreads();
            if (!rev) put();
            if (c0 == middle) __syncthreads();
            if (rev) put();
            if (c0 == middle) __syncthreads();
        } else {
#pragma unroll
            for (int h = 0; h < CH; ++h) {
                if (slot_of[h] >= nc) continue;
                const int left = near(L - c0);
                Tout* yrow = static_cast<Tout*>(g.y) + row0[h] + c0 + loff[h];
                Tout o[T];
#pragma unroll
                for (int i = 0; i < T; ++i) o[i] = from_f32<Tout>(yv[h][i]);
                if (sl * T + T <= left) {
                    __builtin_memcpy(yrow, o, sizeof(o));
                } else {
#pragma unroll
                    for (int i = 0; i < T; ++i)
                        if (sl * T + i < left) yrow[i] = o[i];
                }
            }
        }
    }

    if constexpr (kMode != kFused) {
        if (bad) {
            __threadfence();  // after the stores of the loop above
            walk_positions<T, kPlanes, Tin, Tout, kMode, kZoh>(wv, nullptr);
        }
    } else {
        __syncthreads();
        const float nan = fold_planes<T, kPlanes, Tin, Tout>(g, here, lds);
        // the input planes are no longer read: a word for each wave
        uint32_t* redo = reinterpret_cast<uint32_t*>(lds);
        const bool any = __builtin_amdgcn_ballot_w64(nan != 0.0f) != 0;
        if (lane == 0) redo[wv] = any;
        __syncthreads();
        if (redo[0] | redo[1] | redo[2] | redo[3]) {
            __threadfence();  // after the stores above
#pragma unroll 1
            for (int pass = 0; pass < 2; ++pass) {  // forward directions first
                if (rev == (pass == 1)) walk_positions<T, kPlanes, Tin, Tout, kMode, kZoh>(wv, lds);
                __syncthreads();
            }
            const RowArgs again = args_again();
            fold_planes<T, kPlanes, Tin, Tout>(again, place_of<kMode, kPlanes>(again, wv), lds);
        }
    }
}

// ------------------------------------------------------------------ launch

// LDS of a fused workgroup, at most. Two workgroups a CU or more; a plane that
// leaves room for only one costs less than the merge pass with one or two
// states and more with many (97x101, 768 rows of sequences: N = 1 33 against
// 64 us, with 3072 rows 95 against 167 and N = 8 276 against 220).
constexpr size_t kCuLds = 160 * 1024;
inline size_t fused_lds_limit(int64_t N) { return N <= 2 ? kCuLds : kCuLds / 2; }

size_t fused_lds(int64_t L, int cpw, int T, size_t in_size) {
    return static_cast<size_t>(cpw) * row_len(L, T) * 2 * (in_size + sizeof(float));
}

template <int S, int T, int CH, int NP, typename Tin, typename Tout, int kMode, bool kZoh, bool kN1>
vmb_status launch_rows(const ScanArgs& a, void* y, const void* xt) {
    constexpr int kPlanes = CH * (kWave / S);
    const int64_t per = kMode == kFused ? kPlanes : kPlanes * kRowWaves;
    const int64_t groups = (a.channels + per - 1) / per;
    if (groups > 0x7fffffffLL) return VMB_ERR_UNSUPPORTED;
    const int64_t gy = kMode == kFused ? 1 : a.K;
    const size_t lds = kMode == kFused ? fused_lds(a.L, kPlanes, T, sizeof(Tin)) : 0;
    // a grid has fewer than 2^32 threads in x
    constexpr int64_t kMost = (int64_t{1} << 32) / kRowThreads - 1;
    for (int64_t first = 0; first < groups; first += kMost) {
        const int64_t part = groups - first < kMost ? groups - first : kMost;
        const int64_t n_wg = part * gy * a.batch;
        const RowArgs g{a.u, a.delta, a.A, a.B, a.C, a.D, a.dt_bias, y, xt,
                        int(a.batch), int(a.K), int(a.channels), int(a.N), int(a.H), int(a.W),
                        a.softplus, a.L, int(part), int(first),
                        n_wg <= 0x7fffffffLL ? static_cast<unsigned>(n_wg) : 0u};
        const dim3 grid(static_cast<unsigned>(part), static_cast<unsigned>(gy),
                        static_cast<unsigned>(a.batch));
        hipLaunchKernelGGL((k_full_scan_rows<S, T, CH, NP, Tin, Tout, kMode, kZoh, kN1>), grid,
                           dim3(kRowThreads), lds, a.stream, g);
    }
    return check_launch();
}

// Two recurrences at a time per lane: two channels, which share the B and C
// they read, or two states of one channel (one, with one state). Two channels
// need half the reads from L2 (32 x 56x56, 192 channels, N = 16, fp32 in
// sequence layout: 601 -> 504 us; 32 x 28x28, 384 channels, 2-D 390 -> 296),
// but half the waves: taken when that leaves every SIMD two of them, and in
// the fused form only while LDS still admits four workgroups a CU (32 x 56x56,
// bf16, N = 8: 360 against 322 us).
template <int S, int T, typename Tin, typename Tout, int kMode>
vmb_status launch_np(const ScanArgs& a, void* y, const void* xt) {
    const bool zoh = (a.options & VMB_SCAN_ZOH) != 0;
    constexpr int kCpw = kWave / S;
    const bool two = a.batch * a.K * a.channels >= 2 * kCpw * 2048 &&
                     (kMode != kFused || fused_lds(a.L, 2 * kCpw, T, sizeof(Tin)) <= kCuLds / 4);
    if (a.N == 1) {
        if (zoh) return launch_rows<S, T, 1, 1, Tin, Tout, kMode, true, true>(a, y, xt);
        return two ? launch_rows<S, T, 2, 1, Tin, Tout, kMode, false, true>(a, y, xt)
                   : launch_rows<S, T, 1, 1, Tin, Tout, kMode, false, true>(a, y, xt);
    }
    if (zoh) return launch_rows<S, T, 1, 2, Tin, Tout, kMode, true, false>(a, y, xt);
    return two ? launch_rows<S, T, 2, 1, Tin, Tout, kMode, false, false>(a, y, xt)
               : launch_rows<S, T, 1, 2, Tin, Tout, kMode, false, false>(a, y, xt);
}

// Segment and run length: the shortest pass that holds the sequence (16 lanes
// x 4 positions, 16 x 8, 32 x 8), else a whole wave walking chunks of 512.
template <typename Tin, typename Tout, int kMode>
vmb_status launch_shape(const ScanArgs& a, void* y, const void* xt) {
    if (a.L <= 64) return launch_np<16, 4, Tin, Tout, kMode>(a, y, xt);
    if (a.L <= 128) return launch_np<16, 8, Tin, Tout, kMode>(a, y, xt);
    if (a.L <= 256) return launch_np<32, 8, Tin, Tout, kMode>(a, y, xt);
    return launch_np<64, 8, Tin, Tout, kMode>(a, y, xt);
}

bool fused_fits(const ScanArgs& a) {
    const size_t in = a.in_dt == VMB_F32 ? 4 : 2;
    return a.L <= 16384 && fused_lds(a.L, 1, 8, in) <= fused_lds_limit(a.N);
}

template <typename Tin, typename Tout>
vmb_status dispatch(const ScanArgs& a) {
    if (a.layout == VMB_LAYOUT_SEQ) return launch_shape<Tin, Tout, kSeq>(a, a.y, nullptr);
    if (fused_fits(a)) return launch_shape<Tin, Tout, kFused>(a, a.y, nullptr);
    // planes beyond LDS: per-direction fp32 outputs, then the merge pass; with
    // N = 16 the workspace also has room for column-major plane copies
    const void* xt = nullptr;
    vmb_status st;
    if (full_ws_has_xt(a.batch, a.K, a.channels, a.L, a.N)) {
        void* xtw = static_cast<char*>(a.ws) + full_ws_xt_offset(a.batch, a.K, a.channels, a.L);
        st = launch_transpose_planes(a.u, xtw, a.batch, a.channels, a.H, a.W, a.in_dt, a.stream);
        if (st != VMB_OK) return st;
        xt = xtw;
    }
    st = launch_np<64, 8, Tin, float, kMapRows>(a, a.ws, xt);
    if (st != VMB_OK) return st;
    return launch_cross_merge(a.ws, a.y, a.batch, a.channels, a.H, a.W, VMB_F32, a.out_dt,
                              a.stream);
}

}  // namespace

vmb_status launch_full_rows(const ScanArgs& a) {
    if (a.batch > 65535 || a.K > 65535) return VMB_ERR_UNSUPPORTED;
    if (a.in_dt == VMB_F32) return dispatch<float, float>(a);
    if (a.out_dt == VMB_BF16) return dispatch<bf16_t, bf16_t>(a);
    return dispatch<bf16_t, float>(a);
}

}  // namespace vmb
