// projections.hip -- the selection projections of eq. 6 ahead of the scan.
//
// Appendix A, Mamba paragraph, eq. 6: the selection functions make B, C and
// the timescale depend on the input through linear projections,
//   s_B(u) = Linear_N(u),  s_C(u) = Linear_N(u),
//   s_Delta(u) = Broadcast_D(Linear_1(u)),  Delta = softplus(Parameter + s_Delta(u)).
// Per (batch, direction k) sequence u[d, t] (d over the channels) and with
// the direction's weights W[k] = [R timescale rows; N rows for B; N for C]:
//   x_dbl[r, t]   = sum_d W[k, r, d] u[d, t]            (r < R + 2N)
//   B[n, t]       = x_dbl[R + n, t],  C[n, t] = x_dbl[R + N + n, t]
//   delta[d, t]   = sum_r W_dt[k, d, r] x_dbl[r, t]     (rank R; R = 1 and no W_dt:
//                                                        x_dbl[0, t], the broadcast)
// delta is s_Delta(u): the scan adds the Parameter (dt_bias) and applies softplus.
//
// Both products are dense contractions on the matrix cores. Every wave works
// on its own, from global memory through registers: a lane loads VP
// consecutive positions of a channel row as one vector, and element j of it
// is the operand of column block j, so column c of block j is position
// VP c + j of the wave's 16 VP positions. That permutation of the positions
// makes every load and store of a row one contiguous segment of 16 VP
// elements and, since a column never mixes with another, needs no transpose
// through LDS. The order in which the contraction runs over the
// channels is free as well: a lane group takes the channels whose weights are
// consecutive in memory (one vector load of W).
//   1. x_dbl: steps of 16 (fp32) or 32 (bf16) channels, the next step's u and
//      W loads in flight during a step's products. fp32 inputs take
//      v_mfma_f32_16x16x4f32. bf16 inputs take v_mfma_f32_16x16x32_bf16: u is
//      exact in bf16, W is split into bf16 hi + lo parts (hi the rounded W, lo
//      the rounded remainder), and the two products per row block are exact in
//      fp32, so W is carried to about 2^-17 of itself (far below the bf16
//      rounding of the outputs).
//      The KS waves of a tile take every KS-th step and their sums meet in
//      LDS, added in a fixed order.
//   2. delta: the accumulator of x_dbl row 4 q + v of a block, held by lane
//      group q, is used as it is as the operand of contraction step v (whose
//      four indices are then the rows v, 4 + v, 8 + v, 12 + v), against the
//      four consecutive W_dt[d, 4 q ..] the lane loads as one vector. KS waves
//      take every KS-th block of 16 channels.
// What bounds it (32 x 28x28, 384 channels, rank 12, fp32, 308 MB of u and
// delta): the same tile-wise copy without products takes 72 us (4.3 TB/s; 58 us
// in linear order) and the products 33 us at the fp32 matrix rate; they
// overlap only in part, 93 us (128 with u and W staged in LDS behind two
// barriers per 64 channels, and the low-rank product through LDS). More steps
// in flight (2 or 3) or three or four waves a SIMD measured no faster.
// 32 x 14x14, 768 channels, rank 24, bf16: 103 -> 36 us; 128 x 56x56, 192
// channels, rank 6, bf16: 523 -> 309 us.
// Positions are taken in groups of VP per sequence; the last group of a
// sequence starts at L - VP and forms the positions it shares with the group
// before a second time, to the same bits. 16x16 accumulators: register v of
// lane l is row 4 (l / 16) + v, column l % 16.
//
// The dispatcher deals workgroups to the eight XCDs (each with its own L2)
// round-robin; the 1-D grid is renumbered to give each XCD a contiguous range
// of tiles, so tiles that share a cache line or the weights share an L2.
#include <type_traits>

#include "vmb_internal.h"

namespace vmb {
namespace {

constexpr int kMaxMB = 6;  // 16-row blocks of x_dbl at most (R <= 64, N <= 16)
constexpr int kMaxR = 64;  // timescale rank at most
constexpr int kThreads = 256;
constexpr int kWaves = 4;

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ f32x4 mfma16x16x4(float a, float b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 mfma16x16x32(u32x4 a, u32x4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                   __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

__device__ __forceinline__ uint32_t bf16_bits(float x) { return from_f32<bf16_t>(x).bits; }
__device__ __forceinline__ float bf16_value(uint32_t b) { return __uint_as_float(b << 16); }

// VP consecutive elements of a row
template <typename T, int VP>
struct Vec {
    T v[VP];
};

// channels per step and per lane (a lane group holds a quarter of a step)
template <typename T>
constexpr int step_channels() {
    return sizeof(T) == 4 ? 16 : 32;
}

// registers of one step: u of the lane's channels and W of all row blocks
template <typename T, int MB, int VP>
struct Step {
    static constexpr int kCh = step_channels<T>() / 4;
    Vec<T, VP> u[kCh];
    float w[MB][kCh];
};

// kFlat: sequences shorter than a vector. Positions run on over the batch,
// column c of block j is position 16 j + c of the wave's, each loaded and
// stored by itself (groups is then the number of positions).
template <typename T, int MB, int VP, int KS, bool kFlat>
__global__ __launch_bounds__(kThreads, 2) void k_projections(
    const T* __restrict__ u, const float* __restrict__ W, const float* __restrict__ Wdt,
    T* __restrict__ delta, T* __restrict__ Bo, T* __restrict__ Co, int K, int Dc, int L, int N,
    int R, int64_t groups, int tiles) {
    static_assert(KS == 2 || KS == 4, "two or four waves share a tile");
    constexpr int PW = kWaves / KS;  // tiles per workgroup
    constexpr int kStep = step_channels<T>();
    constexpr int kCh = kStep / 4;
    constexpr int NB = 2;            // step buffers: one step in flight
    constexpr int kRegs = MB * VP;   // accumulators (4 registers each) of a tile
    __shared__ float part[kWaves / 2 * kRegs * 256];

    const int nwg = static_cast<int>(gridDim.x), wg = static_cast<int>(blockIdx.x);
    const int q = nwg / 8, rem = nwg % 8, xcd = wg % 8;
    const int logical = xcd * q + (xcd < rem ? xcd : rem) + wg / 8;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int pw = wv % PW, ks = wv / PW;
    const int wgs_k = (tiles + PW - 1) / PW;  // workgroups per direction
    const int k = logical / wgs_k;
    // (the waves of a tile past the last work on its last position and return
    // after the join)
    const int tile = (logical - k * wgs_k) * PW + pw;
    const int col = lane & 15, kq = lane >> 4;
    const int M = R + 2 * N;  // (M + 15) / 16 == MB
    const size_t l = static_cast<size_t>(L);

    // this lane's VP positions: of one sequence, from tj[0] on, or (kFlat) the
    // position tj[j] of (batch, direction) bkj[j] each
    constexpr int kSeqs = kFlat ? VP : 1;
    size_t bkj[kSeqs];
    int tj[kSeqs];
    size_t at0[kSeqs];  // in channel 0 of u and delta
    bool okj[kSeqs];
    if constexpr (kFlat) {
#pragma unroll
        for (int j = 0; j < VP; ++j) {
            const int64_t p = static_cast<int64_t>(tile) * (16 * VP) + 16 * j + col;
            okj[j] = p < groups;
            const int64_t pc = okj[j] ? p : groups - 1;
            const int64_t b = pc / L;
            tj[j] = static_cast<int>(pc - b * L);
            bkj[j] = static_cast<size_t>(b) * K + k;
        }
    } else {
        const int per_seq = (L + VP - 1) / VP;
        const int64_t gi = static_cast<int64_t>(tile) * 16 + col;
        okj[0] = gi < groups;
        const int64_t gc = okj[0] ? gi : groups - 1;
        const int64_t b = gc / per_seq;
        const int tg = static_cast<int>(gc - b * per_seq) * VP;
        tj[0] = tg + VP <= L ? tg : L - VP;
        bkj[0] = static_cast<size_t>(b) * K + k;
    }
#pragma unroll
    for (int j = 0; j < kSeqs; ++j) at0[j] = bkj[j] * Dc * l + tj[j];
    const bool ok = okj[0];  // the first of them: none where not
    // the positions off elements on from at0 in u, and from at in out
    auto load_at = [&](Vec<T, VP>& v, size_t off) {
        if constexpr (kFlat) {
#pragma unroll
            for (int j = 0; j < VP; ++j) v.v[j] = u[at0[j] + off];
        } else {
            __builtin_memcpy(&v, u + at0[0] + off, sizeof(v));
        }
    };
    auto store_at = [&](T* out, const size_t (&at)[kSeqs], size_t off, const Vec<T, VP>& v) {
        if constexpr (kFlat) {
#pragma unroll
            for (int j = 0; j < VP; ++j)
                if (okj[j]) out[at[j] + off] = v.v[j];
        } else {
            __builtin_memcpy(out + at[0] + off, &v, sizeof(v));
        }
    };

    // 1. x_dbl
    const float* Wk = W + static_cast<size_t>(k) * M * Dc;
    // W row of this lane in each row block (the last block's rows past M repeat one)
    const int m_last = 16 * (MB - 1) + col;
    const float* wlane = Wk + static_cast<size_t>(col) * Dc + kq * kCh;
    const float* wlast = Wk + static_cast<size_t>(m_last < M ? m_last : M - 1) * Dc + kq * kCh;
    auto load = [&](Step<T, MB, VP>& s, int g) {  // a whole step, no branches
        const size_t c0 = static_cast<size_t>(g) * kStep;
        const size_t first = (c0 + kq * kCh) * l;
#pragma unroll
        for (int i = 0; i < kCh; ++i) load_at(s.u[i], first + i * l);
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
            __builtin_memcpy(s.w[mb],
                             (mb + 1 < MB ? wlane + static_cast<size_t>(16 * mb) * Dc : wlast) + c0,
                             sizeof(s.w[mb]));
    };
    // the last Dc % kStep channels: past the end both operands are 0
    auto load_tail = [&](Step<T, MB, VP>& s, int g) {
        const int c0 = g * kStep + kq * kCh;
#pragma unroll
        for (int i = 0; i < kCh; ++i) {
            const int c = c0 + i < Dc ? c0 + i : Dc - 1;
            load_at(s.u[i], static_cast<size_t>(c) * l);
#pragma unroll
            for (int j = 0; j < VP; ++j)
                if (c0 + i >= Dc) s.u[i].v[j] = from_f32<T>(0.0f);
        }
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            const int m = 16 * mb + col;
            const float* wr = Wk + static_cast<size_t>(m < M ? m : M - 1) * Dc;
#pragma unroll
            for (int i = 0; i < kCh; ++i) {
                const float w = wr[c0 + i < Dc ? c0 + i : Dc - 1];
                s.w[mb][i] = c0 + i < Dc ? w : 0.0f;
            }
        }
    };
    f32x4 acc[MB][VP];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int j = 0; j < VP; ++j) acc[mb][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    auto multiply = [&](const Step<T, MB, VP>& s) {
        if constexpr (sizeof(T) == 4) {
#pragma unroll
            for (int i = 0; i < kCh; ++i)
#pragma unroll
                for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                    for (int j = 0; j < VP; ++j)
                        acc[mb][j] = mfma16x16x4(s.w[mb][i], s.u[i].v[j], acc[mb][j]);
        } else {
            u32x4 bv[VP];
#pragma unroll
            for (int j = 0; j < VP; ++j)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    bv[j][i] = s.u[2 * i].v[j].bits |
                               (static_cast<uint32_t>(s.u[2 * i + 1].v[j].bits) << 16);
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) {
                u32x4 hi, lo;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float w0 = s.w[mb][2 * i], w1 = s.w[mb][2 * i + 1];
                    const uint32_t h0 = bf16_bits(w0), h1 = bf16_bits(w1);
                    hi[i] = h0 | (h1 << 16);
                    lo[i] = bf16_bits(w0 - bf16_value(h0)) | (bf16_bits(w1 - bf16_value(h1)) << 16);
                }
#pragma unroll
                for (int j = 0; j < VP; ++j) {
                    acc[mb][j] = mfma16x16x32(hi, bv[j], acc[mb][j]);
                    acc[mb][j] = mfma16x16x32(lo, bv[j], acc[mb][j]);
                }
            }
        }
    };
    // Whole steps ks, ks + KS, ..: NB - 1 of them in flight during a step's
    // products. The loop body is one block without branches, its loads held
    // ahead of the products (the compiler sinks them to their uses otherwise,
    // and waits for all loads where paths join); past the last step the last
    // one is loaded again.
    const int whole = Dc / kStep;
    const int mine = ks < whole ? (whole - ks + KS - 1) / KS : 0;
    if (mine > 0) {
        Step<T, MB, VP> s[NB];
        auto at = [&](int i) { return ks + KS * (i < mine ? i : mine - 1); };
#pragma unroll
        for (int i = 0; i + 1 < NB; ++i) load(s[i], at(i));
        int it = 0;
        for (; it + NB <= mine; it += NB) {
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                load(s[(i + NB - 1) % NB], at(it + i + NB - 1));
                __builtin_amdgcn_sched_barrier(0);
                multiply(s[i]);
            }
        }
#pragma unroll
        for (int i = 0; i + 1 < NB; ++i)
            if (it + i < mine) multiply(s[i]);
    }
    if (Dc % kStep != 0 && whole % KS == ks) {
        Step<T, MB, VP> s;
        load_tail(s, whole);
        multiply(s);
    }
    const int rblocks = (R + 15) / 16;
    // The sums of the tile's waves: the upper half hands its own to the
    // lower, then each wave adds the KS / 2 pair sums for the blocks it
    // goes on with (the timescale rows, and its share of the B and C
    // rows). Half the LDS of one slot a wave.
    constexpr int kHalf = KS / 2;
    auto slot = [&](int w, int mb, int j) {
        return reinterpret_cast<f32x4*>(part + (pw * kHalf + w) * kRegs * 256 +
                                        ((mb * VP + j) * 64 + lane) * 4);
    };
    if (ks >= kHalf) {
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int j = 0; j < VP; ++j) *slot(ks - kHalf, mb, j) = acc[mb][j];
    }
    __syncthreads();
    if (ks < kHalf) {
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int j = 0; j < VP; ++j) *slot(ks, mb, j) += acc[mb][j];
    }
    __syncthreads();
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
        if (mb >= rblocks && mb % KS != ks) continue;
#pragma unroll
        for (int j = 0; j < VP; ++j) {
            f32x4 s = *slot(0, mb, j);
#pragma unroll
            for (int w = 1; w < kHalf; ++w) s += *slot(w, mb, j);
            acc[mb][j] = s;
        }
    }
    if (tile >= tiles) return;

    // B and C rows
    if (ok) {
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            if (mb % KS != ks) continue;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int m = 16 * mb + 4 * kq + v;
                if (m < R || m >= M) continue;
                Vec<T, VP> o;
#pragma unroll
                for (int j = 0; j < VP; ++j) o.v[j] = from_f32<T>(acc[mb][j][v]);
                const int n = m - R;
                size_t at[kSeqs];
#pragma unroll
                for (int j = 0; j < kSeqs; ++j) at[j] = bkj[j] * N * l + tj[j];
                store_at(n < N ? Bo : Co, at, (n < N ? n : n - N) * l, o);
            }
        }
    }

    // 2. delta
    if (Wdt == nullptr) {
        // R = 1, Broadcast_D: every channel takes x_dbl row 0 (register 0 of
        // lane group 0); the lane groups share the channels
        Vec<T, VP> o;
#pragma unroll
        for (int j = 0; j < VP; ++j) o.v[j] = from_f32<T>(__shfl(acc[0][j][0], col, 64));
        if (!ok) return;
        for (int d = 4 * ks + kq; d < Dc; d += 4 * KS)
            store_at(delta, at0, static_cast<size_t>(d) * l, o);
        return;
    }
    constexpr int RB = MB < kMaxR / 16 ? MB : kMaxR / 16;  // blocks that may hold timescale rows
    f32x4 x[RB][VP];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int j = 0; j < VP; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                x[rb][j][v] = 16 * rb + 4 * kq + v < R ? acc[rb][j][v] : 0.0f;
    const float* Wd = Wdt + static_cast<size_t>(k) * Dc * R;
    // Blocks of 16 channels, the next block's weights in flight during the
    // current one's products. kVec: R % 4 == 0, a lane's four weights are one
    // aligned vector, all in or all past the rank (past it, any in-range
    // value: masked before use). kRB: the blocks of timescale rows there are.
    auto channels = [&](auto vec_tag, auto rb_tag) __attribute__((always_inline)) {
        constexpr bool kVec = decltype(vec_tag)::value;
        constexpr int kRB = decltype(rb_tag)::value < RB ? decltype(rb_tag)::value : RB;
        auto load_dt = [&](f32x4 (&a)[kRB], int d0) {
            const int d = d0 + col < Dc ? d0 + col : Dc - 1;
            const float* row = Wd + static_cast<size_t>(d) * R;
#pragma unroll
            for (int rb = 0; rb < kRB; ++rb) {
                const int r = 16 * rb + 4 * kq;
                if constexpr (kVec) {
                    __builtin_memcpy(&a[rb], row + (r < R ? r : 0), 16);
                } else {
#pragma unroll
                    for (int v = 0; v < 4; ++v) a[rb][v] = row[r + v < R ? r + v : 0];
                }
            }
        };
        auto block = [&](const f32x4 (&a)[kRB], int d0) {
            f32x4 o[VP];
#pragma unroll
            for (int j = 0; j < VP; ++j) o[j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int rb = 0; rb < kRB; ++rb) {
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const float w = 16 * rb + 4 * kq + v < R ? a[rb][v] : 0.0f;
#pragma unroll
                    for (int j = 0; j < VP; ++j) o[j] = mfma16x16x4(w, x[rb][j][v], o[j]);
                }
            }
            if (!ok) return;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int d = d0 + 4 * kq + v;
                Vec<T, VP> s;
#pragma unroll
                for (int j = 0; j < VP; ++j) s.v[j] = from_f32<T>(o[j][v]);
                if (d < Dc) store_at(delta, at0, static_cast<size_t>(d) * l, s);
            }
        };
        const int blocks = (Dc + 15) / 16;
        const int mine = ks < blocks ? (blocks - ks + KS - 1) / KS : 0;
        if (mine == 0) return;
        f32x4 a0[kRB], a1[kRB];
        auto at = [&](int i) { return 16 * (ks + KS * (i < mine ? i : mine - 1)); };
        load_dt(a0, at(0));
        int i = 0;
        for (; i + 2 <= mine; i += 2) {
            load_dt(a1, at(i + 1));
            __builtin_amdgcn_sched_barrier(0);
            block(a0, at(i));
            load_dt(a0, at(i + 2));
            __builtin_amdgcn_sched_barrier(0);
            block(a1, at(i + 1));
        }
        if (i < mine) block(a0, at(i));
    };
    auto blocks_of = [&](auto vec_tag) __attribute__((always_inline)) {
        if (rblocks == 1)
            channels(vec_tag, std::integral_constant<int, 1>{});
        else if (rblocks == 2)
            channels(vec_tag, std::integral_constant<int, 2>{});
        else
            channels(vec_tag, std::integral_constant<int, RB>{});
    };
    if ((R & 3) == 0)
        blocks_of(std::true_type{});
    else
        blocks_of(std::false_type{});
}

struct Args {
    const void* u;
    const float *W, *W_dt;
    void *delta, *B, *C;
    int64_t batch;
    int K, Dc, L, N, R;
    hipStream_t s;
};

template <typename T, int MB, int VP, int KS, bool kFlat>
void launch_mb(const Args& a) {
    const int64_t l = a.L, groups = kFlat ? (a.batch * l + VP - 1) / VP : a.batch * ((l + VP - 1) / VP);
    const int64_t tiles = (groups + 15) / 16;
    constexpr int PW = kWaves / KS;
    const int64_t wgs = (tiles + PW - 1) / PW * a.K;
    hipLaunchKernelGGL((k_projections<T, MB, VP, KS, kFlat>), dim3(static_cast<unsigned>(wgs)),
                       dim3(kThreads), 0, a.s, static_cast<const T*>(a.u), a.W, a.W_dt,
                       static_cast<T*>(a.delta), static_cast<T*>(a.B), static_cast<T*>(a.C), a.K,
                       a.Dc, a.L, a.N, a.R, kFlat ? a.batch * l : groups,
                       static_cast<int>(tiles));
}

template <typename T, int VP, int KS, bool kFlat = false>
void launch_vp(const Args& a) {
    switch ((a.R + 2 * a.N + 15) / 16) {
        case 1: return launch_mb<T, 1, VP, KS, kFlat>(a);
        case 2: return launch_mb<T, 2, VP, KS, kFlat>(a);
        case 3: return launch_mb<T, 3, VP, KS, kFlat>(a);
        case 4: return launch_mb<T, 4, VP, KS, kFlat>(a);
        case 5: return launch_mb<T, 5, VP, KS, kFlat>(a);
        default: return launch_mb<T, 6, VP, KS, kFlat>(a);
    }
}

// Tile width and channel split. Measured when they were chosen (us; four waves a
// tile, two, one, or two positions a lane and four waves; since then the
// addressing took 3 to 7% off the fp32 rows), VMamba stages at batch 32:
//   28x28 fp32 rank 12      1568 tiles   100  112  107  111
//   14x14 bf16 rank 24       392 tiles    39   42   68   48
//   7x7 fp32 rank 48         104 tiles    66  122  232   45
//   128 x 56x56 bf16 rank 6  25088 tiles  372  314  312  524
//   2 x 128x512 fp32 rank 6  8192 tiles   217  210  215  252
// so four waves share a tile until the tiles alone fill the chip several
// times over (then two: less to exchange), and tiles get narrower only when
// there are fewer than compute units. Sequences shorter than a vector
// (L < 4): single positions a lane while there are fewer tiles of 64 than
// compute units; from there on tiles over the batch, since single positions
// read W four times as often. Measured (us; single positions, four waves, two):
//   16384 x 3, 192 channels, rank 6    fp32 188 161 163   bf16 211 162 143
//   65536 x 3, 64 channels, N = 8             234 214 242        200 201 178
//   65536 x 1, 96 channels, rank 3            158 136 120        135 113 125
//   4096 x 3, 64 channels, rank 2              20  19  24         19  18  20
template <typename T>
void launch_t(const Args& a) {
    if (a.L < 4) {
        const int64_t tiles = (a.batch * a.L + 63) / 64 * a.K;
        if (tiles < 256) return launch_vp<T, 1, 4>(a);
        if (sizeof(T) == 2 && a.L > 1 && tiles >= 2048) return launch_vp<T, 4, 2, true>(a);
        return launch_vp<T, 4, 4, true>(a);
    }
    const int64_t tiles4 = (a.batch * ((a.L + int64_t{3}) / 4) + 15) / 16 * a.K;
    if (tiles4 < 256) return launch_vp<T, 2, 4>(a);
    if (tiles4 >= 4096) return launch_vp<T, 4, 2>(a);
    launch_vp<T, 4, 4>(a);
}

}  // namespace

vmb_status launch_projections(const void* u, const float* W, const float* W_dt, void* delta,
                              void* B, void* C, int64_t batch, int64_t K, int64_t channels,
                              int64_t L, int64_t N, int64_t R, vmb_dtype dt, hipStream_t s) {
    if (R > kMaxR || R + 2 * N > 16 * kMaxMB || (batch * L + 15) / 16 * K > int64_t{0x7fffffff})
        return VMB_ERR_UNSUPPORTED;
    const Args a{u, W, W_dt, delta, B, C, batch, int(K), int(channels), int(L), int(N), int(R), s};
    if (dt == VMB_F32)
        launch_t<float>(a);
    else
        launch_t<bf16_t>(a);
    return check_launch();
}

}  // namespace vmb
