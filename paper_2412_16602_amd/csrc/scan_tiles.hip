// scan_tiles.hip -- full selective scan for grids with many channel rows
// (the batched VMamba stages), N = 16.
//
// Same recurrence as scan_full.hip (Appendix A: eq. 3, eq. 4 first line,
// eq. 6): h_t = exp(Delta_t A_n) h_{t-1} + Delta_t B_t u_t from h_{-1} = 0,
// y_t = sum_n C_t h_t + D u_t, Delta = softplus(delta + dt_bias).
//
// Work decomposition. A workgroup owns 64 channels of one (batch, direction)
// and walks the sequence in tiles of 16 positions. Lanes are channels; the
// 16 states are split over the four waves, four each, so every lane runs four
// independent recurrences straight along the sequence: no cross-lane scan,
// no re-walk. Per (channel, state, position): mul, exp2, mul, fma, fma.
//   - B[n, t] and C[n, t] are the same for every channel of a direction, so a
//     wave's four rows are wave-uniform: they are read with scalar loads into
//     SGPRs and used as the scalar operand of the VALU instructions.
//   - delta and u arrive in coalesced row pieces (each thread 4 positions of
//     one channel), are discretized once per (channel, position) by the
//     thread that loaded them (Delta log2 e, Delta u, D u) and transposed
//     through LDS for the channel-per-lane walk.
//   - Each wave's partial output (its four states' C h) goes back through LDS
//     and the loading threads add the four partials and D u, then store y
//     with row-contiguous vectors.
// Two workgroup barriers per tile; the next tile's delta / u loads, and one
// load per B / C row segment that brings those lines into L2, are in flight
// while the current tile is scanned; they are kept as loaded and converted
// where they are used, since a conversion beside a load waits for it.
//
// What bounds it: instruction issue. Per element a multiply (2.5 cycles a wave
// on its SIMD), an exp2 (8.3), a multiply and an fma with a scalar operand
// (4.3 each; 2.5-2.8 without) and an fma (2.8): 22 of the 36 measured at 128 x
// 28x28, 384 channels, fp32. 128 x 56x56, 192 channels, bf16, 2-D step: 1634 us
// with conversions beside the loads and one wait per half tile for B and C,
// 1480 us without (fp32: unchanged, 166 us at 32 x 28x28, sequence layout), and
// 1460 and 163 us with a select in place of a divergent branch around each
// position's softplus.
//
// Workgroups are numbered so that those sharing a (batch, direction), and
// therefore B and C, land on the same XCD and its L2.

#include "vmb_internal.h"

namespace vmb {
namespace {

constexpr int kWave = 64;
constexpr int kStates = 16;
constexpr int kTileWaves = 4;                     // four states per wave (eight waves of two: no faster)
constexpr int kTileThreads = kTileWaves * kWave;  // 256
constexpr int kTP = 16;                           // positions per tile
constexpr int kStride = kTP + 1;                  // LDS row stride (words): conflict-free columns

// P consecutive elements of a row as they lie in memory: one vector (of any
// element alignment), converted where it is used, so that nothing waits for
// it before.
template <typename Tin, int P>
struct Piece {
    uint32_t w[P * static_cast<int>(sizeof(Tin)) / 4];
};
template <int P>
__device__ __forceinline__ float piece_at(const Piece<float, P>& r, int e) {
    return __uint_as_float(r.w[e]);
}
template <int P>
__device__ __forceinline__ float piece_at(const Piece<bf16_t, P>& r, int e) {
    return __uint_as_float((e & 1) ? r.w[e / 2] & 0xffff0000u : r.w[e / 2] << 16);
}
template <bool kNt, typename Tout, int P>
__device__ __forceinline__ void store_piece(Tout* p, const float (&v)[P]) {
    struct alignas(P * sizeof(Tout)) Out {
        Tout e[P];
    } o;
#pragma unroll
    for (int e = 0; e < P; ++e) o.e[e] = from_f32<Tout>(v[e]);
    if constexpr (kNt)
        store_out<true>(reinterpret_cast<Out*>(p), o);
    else
        __builtin_memcpy(p, &o, sizeof(o));
}

// Four consecutive positions of a wave's S B rows and S C rows, as they lie in
// memory (scalar loads of whole 32-bit words: bf16 rows have even length,
// and quarters start at even positions).
template <typename Tin, int S>
struct Quarter {
    static constexpr int kWords = static_cast<int>(sizeof(Tin));  // 4 elements of a row
    uint32_t b[S][kWords], c[S][kWords];
};
template <typename Tin>
__device__ __forceinline__ float word_value(const uint32_t* w, int e);
template <>
__device__ __forceinline__ float word_value<float>(const uint32_t* w, int e) {
    return __uint_as_float(w[e]);
}
template <>
__device__ __forceinline__ float word_value<bf16_t>(const uint32_t* w, int e) {
    return __uint_as_float((e & 1) ? w[e / 2] & 0xffff0000u : w[e / 2] << 16);
}

// Wait for this wave's scalar loads and LDS operations (lgkmcnt(0), other
// counters untouched).
__device__ __forceinline__ void wait_lgkm() { __builtin_amdgcn_s_waitcnt(0xc07f); }

template <typename Tin, typename Tout, bool kTwoD, bool kZoh, bool kNt>
__global__ __launch_bounds__(kTileThreads) void k_full_scan_tiles(
    const Tin* __restrict__ u, const Tin* __restrict__ delta, const float* __restrict__ A,
    const Tin* __restrict__ Bm, const Tin* __restrict__ Cm, const float* __restrict__ D,
    const float* __restrict__ dt_bias, Tout* __restrict__ y, const Tin* __restrict__ xt, int K,
    int Dc, int L, int H, int W, int softplus, int n_cg, int n_wg) {
    constexpr int N = kStates;
    constexpr int S = N / kTileWaves;              // states per wave
    constexpr int P = kWave * kTP / kTileThreads;  // positions a thread loads and stores
    constexpr int kPieces = kTP / P;               // threads per row
    __shared__ float s_dl2[kWave][kStride];               // Delta * log2 e
    __shared__ float s_du[kWave][kStride];                // Delta * u
    __shared__ float s_y[kTileWaves][kWave][kStride];     // per wave: its states' C h
    __shared__ float s_u[kZoh ? kWave : 1][kStride];      // u itself (zero-order-hold B only)

    // XCD-aware numbering: hardware places workgroup i on XCD i % 8
    const int bid = blockIdx.x;
    const int per = n_wg / 8, rem = n_wg % 8;
    const int xcd = bid % 8, slot = bid / 8;
    const int logical = xcd < rem ? xcd * (per + 1) + slot : rem * (per + 1) + (xcd - rem) * per + slot;
    const int cg = logical % n_cg;
    const int bk = logical / n_cg;  // b * K + k
    const int k = bk % K;
    const int b = bk / K;
    const int d0 = cg * kWave;

    const int tid = threadIdx.x;
    const int lane = tid % kWave;
    const int wv = __builtin_amdgcn_readfirstlane(tid / kWave);
    const bool sp = softplus != 0;

    // Loader role: row lr (channel d0 + lr), positions P lq .. P lq + P - 1 of each tile.
    const int lr = tid / kPieces, lq = tid % kPieces;
    const bool ld_ok = d0 + lr < Dc;
    const int ld_d = ld_ok ? d0 + lr : Dc - 1;  // rows past the end repeat a valid one, unstored
    const int ld_c = k * Dc + ld_d;
    const float ld_bias = dt_bias ? dt_bias[ld_c] : 0.0f;
    const float ld_skip = D ? D[ld_c] : 0.0f;
    const size_t ld_row = (static_cast<size_t>(bk) * Dc + ld_d) * static_cast<size_t>(L);
    const Tin* drow = delta + ld_row;
    const Tin* urow = kTwoD ? u + (static_cast<size_t>(b) * Dc + ld_d) * L : u + ld_row;
    // 2-D layout: direction k's sequence is the plane read row-major (k even)
    // or column-major (k odd: the transposed copy xt when given), forwards
    // for k < 2 and backwards for k >= 2
    const Tin* srow = (kTwoD && (k & 1) && xt) ? xt + (static_cast<size_t>(b) * Dc + ld_d) * L : urow;
    const bool gather = kTwoD && (k & 1) && !xt;
    Tout* yrow = y + ld_row;
    // Scan role: lane = channel d0 + lane, states S wv .. S wv + S - 1.
    const int sd = d0 + lane < Dc ? d0 + lane : Dc - 1;
    const int sc = k * Dc + sd;
    float an[S], h[S], inv_a[S];
#pragma unroll
    for (int j = 0; j < S; ++j) {
        an[j] = A[static_cast<size_t>(sc) * N + S * wv + j];
        inv_a[j] = kZoh ? 1.0f / an[j] : 0.0f;
        h[j] = 0.0f;
    }
    // the wave's B and C rows: one base each, rows L elements apart
    const size_t r0 = (static_cast<size_t>(bk) * N + S * wv) * static_cast<size_t>(L);
    const Tin* bbase = Bm + r0;
    const Tin* cbase = Cm + r0;

    // Tile j covers positions [ts, ts + 16) with ts = 16 j, except the last,
    // which starts at L - 16 (L >= 16) so that every tile is whole: its
    // positions below 16 j were done by the previous tile and are run here
    // as identity steps (Delta = 0: a = 1, b = 0) and not stored again.
    const int ntiles = (L + kTP - 1) / kTP;
    auto tile_start = [&](int tile) { return tile * kTP + kTP <= L ? tile * kTP : L - kTP; };
    Piece<Tin, P> dv, uv;
    const bool reversed = kTwoD && !gather && k >= 2;  // uv holds the piece back to front
    auto load_tile = [&](int tile) {
        const int t = tile_start(tile) + P * lq;
        __builtin_memcpy(&dv, drow + t, sizeof(dv));
        if constexpr (kTwoD) {
            if (gather) {
                Tin e[P];
#pragma unroll
                for (int i = 0; i < P; ++i) e[i] = urow[pixel_of(k, t + i, H, W)];
                __builtin_memcpy(&uv, e, sizeof(uv));
            } else {
                __builtin_memcpy(&uv, srow + (k < 2 ? t : L - P - t), sizeof(uv));
            }
        } else {
            __builtin_memcpy(&uv, urow + t, sizeof(uv));
        }
    };
    load_tile(0);
    // L2 prefetch of the next tile's B and C segments (16 + 16 rows of the
    // direction, one line each), so that the scan's scalar loads of them do
    // not wait for HBM: threads 0..31 each touch one row and hold the value
    // until step 4.
    const Tin* pf_row = (tid < 16 ? Bm : Cm) +
                        (static_cast<size_t>(bk) * N + (tid & 15)) * static_cast<size_t>(L);
    uint32_t pf = 0;  // raw bits: a conversion would wait for the load
    Quarter<Tin, S> bc[2];
    auto load_bc = [&](Quarter<Tin, S>& r, int off) {
        constexpr int kPer = 4 / static_cast<int>(sizeof(Tin));  // elements per word
        // opaque: the quarters' loads are not merged into wider ones, which
        // would all be needed (and held) at once
        unsigned first = static_cast<unsigned>(off) / kPer;
        asm volatile("" : "+s"(first));
        const uint32_t* bq = reinterpret_cast<const uint32_t*>(bbase) + first;
        const uint32_t* cq = reinterpret_cast<const uint32_t*>(cbase) + first;
        const unsigned words = static_cast<unsigned>(L) / kPer;  // of a row
#pragma unroll
        for (int j = 0; j < S; ++j) {
            const uint32_t* bw = bq + static_cast<size_t>(j) * words;
            const uint32_t* cw = cq + static_cast<size_t>(j) * words;
#pragma unroll
            for (int w = 0; w < Quarter<Tin, S>::kWords; ++w) {
                r.b[j][w] = bw[w];
                r.c[j][w] = cw[w];
            }
        }
    };
    load_bc(bc[0], tile_start(0));

    for (int tile = 0; tile < ntiles; ++tile) {
        const int t0 = tile_start(tile);
        const int tnew = tile * kTP;  // positions below tnew belong to the previous tile
        // 1. discretize this thread's P positions
        float skip[P];
        {
            const int t = t0 + P * lq;
            // one uniform branch and a select, no branch per position: the
            // positions' softplus chains interleave
            float step[P];
#pragma unroll
            for (int e = 0; e < P; ++e) step[e] = piece_at<P>(dv, e) + ld_bias;
            if (sp) {
#pragma unroll
                for (int e = 0; e < P; ++e) step[e] = timescale(step[e], true);
            }
#pragma unroll
            for (int e = 0; e < P; ++e) {
                const float ut = reversed ? piece_at<P>(uv, P - 1 - e) : piece_at<P>(uv, e);
                const float dl = t + e >= tnew ? step[e] : 0.0f;
                s_dl2[lr][P * lq + e] = dl * kLog2e;
                s_du[lr][P * lq + e] = dl * ut;
                if constexpr (kZoh) s_u[lr][P * lq + e] = ut;
                skip[e] = ld_skip * ut;
            }
        }
        __syncthreads();
        // 2. the next tile's delta / u (and its B, C lines), in flight during the scan
        if (tile + 1 < ntiles) {
            load_tile(tile + 1);
            if (tid < 2 * N) {
                const Tin* line = pf_row + tile_start(tile + 1);
                if constexpr (sizeof(Tin) == 4)
                    pf = *reinterpret_cast<const uint32_t*>(line);
                else
                    pf = *reinterpret_cast<const uint16_t*>(line);
            }
        }
        // 3. scan the tile: S recurrences per lane, straight along the
        //    positions, in quarters of 4. Scalar loads complete out of order,
        //    so every wait is for all of them (and for LDS, which counts with
        //    them): a quarter's B, C, Delta and Delta u are waited for once,
        //    before the next quarter's are requested, and those are in flight
        //    during its arithmetic (the first quarter of the next tile's B
        //    and C during the last one's).
        float yp[kTP], xd[2][4], xu[2][4], xi[2][4];
        auto read_lds = [&](int q) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                xd[q & 1][e] = s_dl2[lane][4 * q + e];
                xu[q & 1][e] = s_du[lane][4 * q + e];
                xi[q & 1][e] = kZoh ? s_u[lane][4 * q + e] : 0.0f;
            }
        };
        read_lds(0);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            wait_lgkm();
            __builtin_amdgcn_sched_barrier(0);
            if (q < 3) {
                load_bc(bc[(q + 1) & 1], t0 + 4 * (q + 1));
                read_lds(q + 1);
            } else {
                load_bc(bc[0], tile_start(tile + 1 < ntiles ? tile + 1 : tile));
            }
            __builtin_amdgcn_sched_barrier(0);
            const Quarter<Tin, S>& cur = bc[q & 1];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float dl2 = xd[q & 1][e], du = xu[q & 1][e], ui = xi[q & 1][e];
                float acc = 0.0f;
#pragma unroll
                for (int j = 0; j < S; ++j) {
                    const float x2 = dl2 * an[j];
                    const float a = fast_exp2(x2);
                    const float qb = kZoh ? zoh_q(x2, a, du, ui, inv_a[j]) : du;
                    h[j] = __builtin_fmaf(a, h[j], qb * word_value<Tin>(cur.b[j], e));
                    acc = __builtin_fmaf(word_value<Tin>(cur.c[j], e), h[j], acc);
                }
                yp[4 * q + e] = acc;
            }
        }
#pragma unroll
        for (int i = 0; i < kTP; ++i) s_y[wv][lane][i] = yp[i];
        __syncthreads();
        // 4. y = D u + the four waves' partial sums, stored row-contiguous
        //    (a piece that straddles the previous tile stores its new part).
        //    The next tile's loads are waited for here, ahead of the stores:
        //    vector-memory operations retire in order, and waited for after
        //    them they would wait for the stores as well.
#pragma unroll
        for (uint32_t& x : dv.w) asm volatile("" : "+v"(x));
#pragma unroll
        for (uint32_t& x : uv.w) asm volatile("" : "+v"(x));
        asm volatile("" : "+v"(pf));
        {
            const int t = t0 + P * lq;
            float o[P];
#pragma unroll
            for (int e = 0; e < P; ++e) {
                const int i = P * lq + e;
                float part[kTileWaves];  // summed in pairs, in wave order
#pragma unroll
                for (int w = 0; w < kTileWaves; ++w) part[w] = s_y[w][lr][i];
#pragma unroll
                for (int n = kTileWaves; n > 1; n /= 2)
#pragma unroll
                    for (int w = 0; w < n / 2; ++w) part[w] = part[2 * w] + part[2 * w + 1];
                o[e] = skip[e] + part[0];
            }
            if (ld_ok) {
                if (t >= tnew) {
                    store_piece<kNt>(yrow + t, o);
                } else {
#pragma unroll
                    for (int e = 0; e < P; ++e)
                        if (t + e >= tnew) yrow[t + e] = from_f32<Tout>(o[e]);
                }
            }
        }
    }
}

template <typename Tin, typename Tout, bool kTwoD, bool kZoh, bool kNt>
void launch_tiles_kernel(const ScanArgs& a, Tout* y, const void* xt, int n_cg, int n_wg) {
    hipLaunchKernelGGL((k_full_scan_tiles<Tin, Tout, kTwoD, kZoh, kNt>),
                       dim3(static_cast<unsigned>(n_wg)), dim3(kTileThreads), 0, a.stream,
                       static_cast<const Tin*>(a.u), static_cast<const Tin*>(a.delta), a.A,
                       static_cast<const Tin*>(a.B), static_cast<const Tin*>(a.C), a.D, a.dt_bias,
                       y, static_cast<const Tin*>(xt), int(a.K), int(a.channels), int(a.L),
                       int(a.H), int(a.W), a.softplus, n_cg, n_wg);
}

template <typename Tin, typename Tout, bool kTwoD, bool kZoh>
vmb_status launch_tiles_zoh(const ScanArgs& a, Tout* y, const void* xt) {
    const int n_cg = int((a.channels + kWave - 1) / kWave);
    const long long n_wg = static_cast<long long>(n_cg) * a.K * a.batch;
    if (n_wg > 0x7fffffffLL) return VMB_ERR_UNSUPPORTED;
    // non-temporal output stores for rows of whole cache lines
    const bool nt = whole_lines(a.L, sizeof(Tout));
    const int g = int(n_wg);
    if (nt)
        launch_tiles_kernel<Tin, Tout, kTwoD, kZoh, true>(a, y, xt, n_cg, g);
    else
        launch_tiles_kernel<Tin, Tout, kTwoD, kZoh, false>(a, y, xt, n_cg, g);
    return check_launch();
}

template <typename Tin, typename Tout, bool kTwoD>
vmb_status launch_tiles_impl(const ScanArgs& a, Tout* y, const void* xt) {
    return (a.options & VMB_SCAN_ZOH) ? launch_tiles_zoh<Tin, Tout, kTwoD, true>(a, y, xt)
                                      : launch_tiles_zoh<Tin, Tout, kTwoD, false>(a, y, xt);
}

}  // namespace

// Whether the tile kernel takes this shape at all (N = 16, whole tiles; bf16
// rows of even length): the zero-order-hold option runs here whatever the
// number of rows.
bool tiles_take(const ScanArgs& a) {
    return a.N == 16 && a.L >= kTP && !(a.in_dt == VMB_BF16 && (a.L % 2) != 0);
}

// Many channel rows (each sequence's channels split into 64-channel
// workgroups still give several waves per SIMD), N = 16, L >= 16; bf16 rows
// need an even length for the word-wise scalar reads of B and C.
bool use_tiles_full(const ScanArgs& a) {
    if (a.N != 16) return false;
    if (a.L < kTP) return false;  // the last tile starts at L - 16
    if (a.in_dt == VMB_BF16 && (a.L % 2) != 0) return false;
    const int64_t rows = a.batch * a.K * a.channels;
    return rows >= kTilesMinRows;
}

vmb_status launch_full_tiles(const ScanArgs& a, void* y_seq, const void* xt) {
    const bool two_d = a.layout == VMB_LAYOUT_2D;
    if (a.in_dt == VMB_F32)
        return two_d ? launch_tiles_impl<float, float, true>(a, static_cast<float*>(y_seq), xt)
                     : launch_tiles_impl<float, float, false>(a, static_cast<float*>(y_seq), xt);
    if (two_d) return launch_tiles_impl<bf16_t, float, true>(a, static_cast<float*>(y_seq), xt);
    if (a.out_dt == VMB_BF16)
        return launch_tiles_impl<bf16_t, bf16_t, false>(a, static_cast<bf16_t*>(y_seq), xt);
    return launch_tiles_impl<bf16_t, float, false>(a, static_cast<float*>(y_seq), xt);
}

}  // namespace vmb
