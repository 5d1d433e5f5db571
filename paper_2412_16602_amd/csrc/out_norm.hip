// out_norm.hip -- the step after the cross-merge in VMamba's SS2D block: a
// layer normalisation over the channels of each pixel and the SiLU gate.
// (The paper's text stops at the merge; this follows the public VMamba
// block that the paper's models are built from.)
//
// Per pixel p of image b, over the channels d of y[b, d, p] (the 2-D layout):
//   mu    = mean_d y,   var = mean_d (y - mu)^2   (biased)
//   out   = (y - mu) / sqrt(var + eps) * gamma[d] + beta[d]
//   out  *= z / (1 + exp(-z))                     (when z is given)
//
// Pixels are flattened over (batch, p): a workgroup owns PX consecutive
// flattened pixels and its 1024 threads are PX pixels x 1024 / PX channel
// groups (channel d belongs to group d % groups), so every load covers PX
// consecutive pixels of 64 / PX channel rows: PX = 16 for fp32 and 32 for
// bf16 (64-byte row segments either way), halved down to a quarter while the
// grid has fewer than 512 workgroups and every thread keeps four channels
// (short maps: 7x7 at batch 32 has 1568 pixels of 1536 channels). A thread loads all of its
// channels' y and z at once into registers (up to J = 32 each), so the whole
// tensor is in flight and HBM is read once; the mean and the centred sum of
// squares (exact in fp32 for any offset of the mean) are then formed from
// the registers. Wider channel counts stream the channels three times (the
// second and third reads from cache). The group sums are added across each
// wave by shuffles, then the waves' sums in LDS in wave order
// (deterministic). As in the projections, the 1-D grid is dealt to the XCDs
// in contiguous ranges of tiles, so neighbouring tiles, which share the
// 128-byte lines of a channel row, read them through one L2.
#include "vmb_internal.h"

namespace vmb {
namespace {

constexpr int kThreads = 1024;

// Sum of v over the channel groups of this thread's pixel, in a fixed order:
// a wave holds 64 / PX groups of the same PX pixels (lane l: pixel l % PX),
// which are first added across the wave (xor shuffles over the lane bits
// above the pixel's), then the waves' sums in wave order.
template <int PX>
__device__ __forceinline__ float group_total(float (*red)[PX + 1], float* tot, float v, int px,
                                             int grp) {
    constexpr int kWave = 64, kWaves = kThreads / kWave;
#pragma unroll
    for (int m = PX; m < kWave; m *= 2) v += __shfl_xor(v, m, kWave);
    const int lane = threadIdx.x % kWave, wv = threadIdx.x / kWave;
    if (lane < PX) red[wv][px] = v;
    __syncthreads();
    if (grp == 0) {
        float t = 0.0f;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) t += red[w][px];
        tot[px] = t;
    }
    __syncthreads();
    return tot[px];
}

// J > 0: a thread's channels grp + 64 j (j < J) held in registers; J == 0:
// streamed.
template <typename T, int J, int PX>
__global__ __launch_bounds__(kThreads) void k_out_norm(const T* __restrict__ y,
                                                       const T* __restrict__ z,
                                                       const float* __restrict__ gamma,
                                                       const float* __restrict__ beta, float eps,
                                                       T* __restrict__ out, int Dc, int P,
                                                       int64_t pixels) {
    constexpr int kPx = PX, kGroups = kThreads / PX;
    __shared__ float red[kGroups][kPx + 1];
    __shared__ float tot[kPx];
    const int nwg = static_cast<int>(gridDim.x), wg = static_cast<int>(blockIdx.x);
    const int q = nwg / 8, rem = nwg % 8, xcd = wg % 8;
    const int tile = xcd * q + (xcd < rem ? xcd : rem) + wg / 8;
    const int px = threadIdx.x % kPx, grp = threadIdx.x / kPx;
    const int64_t p = static_cast<int64_t>(tile) * kPx + px;
    const bool ok = p < pixels;
    const int64_t pc = ok ? p : 0;  // clamped: loads stay in bounds
    const int64_t b = pc / P;
    const size_t base = static_cast<size_t>(b) * Dc * P + static_cast<size_t>(pc - b * P);
    const size_t pstride = static_cast<size_t>(P);
    const float inv_dc = 1.0f / static_cast<float>(Dc);

    auto finish = [&](int d, float v, float zv, float mu, float rstd) {
        float o = (v - mu) * rstd;
        if (gamma) o *= gamma[d];
        if (beta) o += beta[d];
        if (z) o *= zv / (1.0f + __expf(-zv));
        out[base + d * pstride] = from_f32<T>(o);
    };

    if constexpr (J > 0) {
        // raw values, converted at use: a conversion next to its load (or a
        // test of z per element) would make each load wait for the last
        T yr[J], zr[J];
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int d = grp + kGroups * j;
            yr[j] = y[base + static_cast<size_t>(d < Dc ? d : 0) * pstride];
        }
        if (z) {
#pragma unroll
            for (int j = 0; j < J; ++j) {
                const int d = grp + kGroups * j;
                zr[j] = z[base + static_cast<size_t>(d < Dc ? d : 0) * pstride];
            }
        }
        float yv[J];
#pragma unroll
        for (int j = 0; j < J; ++j) yv[j] = to_f32(yr[j]);
        float s = 0.0f;
#pragma unroll
        for (int j = 0; j < J; ++j)
            if (grp + kGroups * j < Dc) s += yv[j];
        const float mu = group_total<PX>(red, tot, s, px, grp) * inv_dc;
        float s2 = 0.0f;
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const float c = yv[j] - mu;
            if (grp + kGroups * j < Dc) s2 = __builtin_fmaf(c, c, s2);
        }
        const float rstd = 1.0f / sqrtf(group_total<PX>(red, tot, s2, px, grp) * inv_dc + eps);
        if (!ok) return;
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int d = grp + kGroups * j;
            if (d < Dc) finish(d, yv[j], z ? to_f32(zr[j]) : 0.0f, mu, rstd);
        }
    } else {
        float s = 0.0f;
#pragma unroll 8
        for (int d = grp; d < Dc; d += kGroups) s += to_f32(y[base + d * pstride]);
        const float mu = group_total<PX>(red, tot, s, px, grp) * inv_dc;
        float s2 = 0.0f;
#pragma unroll 8
        for (int d = grp; d < Dc; d += kGroups) {
            const float c = to_f32(y[base + d * pstride]) - mu;
            s2 = __builtin_fmaf(c, c, s2);
        }
        const float rstd = 1.0f / sqrtf(group_total<PX>(red, tot, s2, px, grp) * inv_dc + eps);
        if (!ok) return;
#pragma unroll 4
        for (int d = grp; d < Dc; d += kGroups) {
            const size_t off = base + d * pstride;
            finish(d, to_f32(y[off]), z ? to_f32(z[off]) : 0.0f, mu, rstd);
        }
    }
}

// The same with a 16-byte vector of consecutive pixels a lane (V = 4 fp32, 8
// bf16): kLanes lanes cover 8 of them, one 128-byte segment of a channel row
// (4: half of one), 64 channel groups, J channels a thread, all of a thread's
// y and z loads in flight at once. Bound by HBM: 128 x 56x56, 192 channels,
// bf16: 187 us with one pixel a lane (32- to 64-byte segments), 126 with
// vectors (3.7 TB/s); 32 x 56x56, fp32 77 -> 54 (4.3 TB/s); 32 x 28x28, 384
// channels 36 -> 30.5. An image's pixels are taken in groups of V; its last group starts at
// P - V and forms the pixels it shares with the one before a second time, to
// the same bits.
constexpr int kVecGroups = 64;
template <typename T>
constexpr int vec_pixels() {
    return 16 / static_cast<int>(sizeof(T));
}
template <typename T, int J, int kLanes>
__global__ __launch_bounds__(kVecGroups* kLanes) void k_out_norm_vec(
    const T* __restrict__ y, const T* __restrict__ z, const float* __restrict__ gamma,
    const float* __restrict__ beta, float eps, T* __restrict__ out, int Dc, int P,
    int64_t vectors) {
    constexpr int V = vec_pixels<T>();
    constexpr int kWave = 64, kWaves = kVecGroups * kLanes / kWave;
    struct Vec {
        T v[V];
    };
    __shared__ __align__(16) float red[2][kWaves][kLanes][V];
    const int nwg = static_cast<int>(gridDim.x), wg = static_cast<int>(blockIdx.x);
    const int q = nwg / 8, rem = nwg % 8, xcd = wg % 8;
    const int tile = xcd * q + (xcd < rem ? xcd : rem) + wg / 8;
    const int px = threadIdx.x % kLanes, grp = threadIdx.x / kLanes;
    const int lane = threadIdx.x % kWave, wv = threadIdx.x / kWave;
    const int per = (P + V - 1) / V;  // groups per image
    const int64_t g = static_cast<int64_t>(tile) * kLanes + px;
    const bool ok = g < vectors;
    const int64_t gc = ok ? g : vectors - 1;
    const int64_t b = gc / per;
    const int p0 = V * static_cast<int>(gc - b * per);
    const size_t base = static_cast<size_t>(b) * Dc * P + (p0 + V <= P ? p0 : P - V);
    const float inv_dc = 1.0f / static_cast<float>(Dc);

    // raw values, converted at use: a conversion next to its load would make
    // each load wait for the last; rows past the last channel repeat it
    Vec yr[J], zr[J];
#pragma unroll
    for (int j = 0; j < J; ++j) {
        const int d = grp + kVecGroups * j;
        __builtin_memcpy(&yr[j], y + base + static_cast<size_t>(d < Dc ? d : Dc - 1) * P,
                         sizeof(Vec));
    }
    if (z) {
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int d = grp + kVecGroups * j;
            __builtin_memcpy(&zr[j], z + base + static_cast<size_t>(d < Dc ? d : Dc - 1) * P,
                             sizeof(Vec));
        }
    }
    // sums over the channel groups: across the wave by shuffles, then the
    // waves' sums in wave order
    auto total = [&](float (&s)[V], int buf) {
#pragma unroll
        for (int m = kLanes; m < kWave; m *= 2)
#pragma unroll
            for (int i = 0; i < V; ++i) s[i] += __shfl_xor(s[i], m, kWave);
        if (lane < kLanes)
#pragma unroll
            for (int i = 0; i < V; ++i) red[buf][wv][px][i] = s[i];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < V; ++i) s[i] = 0.0f;
#pragma unroll 2
        for (int w = 0; w < kWaves; ++w)
#pragma unroll
            for (int i = 0; i < V; ++i) s[i] += red[buf][w][px][i];
    };
    float mu[V], rstd[V];
#pragma unroll
    for (int i = 0; i < V; ++i) mu[i] = rstd[i] = 0.0f;
#pragma unroll
    for (int j = 0; j < J; ++j)
        if (grp + kVecGroups * j < Dc) {
#pragma unroll
            for (int i = 0; i < V; ++i) mu[i] += to_f32(yr[j].v[i]);
        }
    total(mu, 0);
#pragma unroll
    for (int i = 0; i < V; ++i) mu[i] *= inv_dc;
#pragma unroll
    for (int j = 0; j < J; ++j)
        if (grp + kVecGroups * j < Dc) {
#pragma unroll
            for (int i = 0; i < V; ++i) {
                const float c = to_f32(yr[j].v[i]) - mu[i];
                rstd[i] = __builtin_fmaf(c, c, rstd[i]);
            }
        }
    total(rstd, 1);
#pragma unroll
    for (int i = 0; i < V; ++i) rstd[i] = 1.0f / sqrtf(rstd[i] * inv_dc + eps);
    if (!ok) return;
#pragma unroll
    for (int j = 0; j < J; ++j) {
        const int d = grp + kVecGroups * j;
        if (d >= Dc) break;
        const float ga = gamma ? gamma[d] : 1.0f, be = beta ? beta[d] : 0.0f;
        Vec o;
#pragma unroll
        for (int i = 0; i < V; ++i) {
            float v = (to_f32(yr[j].v[i]) - mu[i]) * rstd[i];
            if (gamma) v *= ga;
            if (beta) v += be;
            if (z) {
                const float zv = to_f32(zr[j].v[i]);
                v *= zv / (1.0f + __expf(-zv));
            }
            o.v[i] = from_f32<T>(v);
        }
        __builtin_memcpy(out + base + static_cast<size_t>(d) * P, &o, sizeof(o));
    }
}

// Channels a thread can hold (8 registers of y and z each).
constexpr int kVecMaxJ = 8;

template <typename T>
void launch_vec(hipStream_t s, const void* y, const void* z, const float* gamma,
                const float* beta, float eps, void* out, int Dc, int P, int64_t vectors) {
    const T* yy = static_cast<const T*>(y);
    const T* zz = static_cast<const T*>(z);
    T* oo = static_cast<T*>(out);
    auto go = [&](auto kernel, int lanes) {
        hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>((vectors + lanes - 1) / lanes)),
                           dim3(kVecGroups * lanes), 0, s, yy, zz, gamma, beta, eps, oo, Dc, P,
                           vectors);
    };
    // from 6 channels a thread the registers leave room for two of the wide
    // workgroups a CU; half as wide, four or five fit and the grid ends more
    // evenly (24 x 28x28, 384 channels 24 -> 19 us; at 3 channels 2% slower)
    switch ((Dc + kVecGroups - 1) / kVecGroups) {
        case 1: return go(k_out_norm_vec<T, 1, 8>, 8);
        case 2: return go(k_out_norm_vec<T, 2, 8>, 8);
        case 3: return go(k_out_norm_vec<T, 3, 8>, 8);
        case 4: return go(k_out_norm_vec<T, 4, 8>, 8);
        case 5: return go(k_out_norm_vec<T, 5, 8>, 8);
        case 6: return go(k_out_norm_vec<T, 6, 4>, 4);
        case 7: return go(k_out_norm_vec<T, 7, 4>, 4);
        default: return go(k_out_norm_vec<T, 8, 4>, 4);
    }
}

template <typename T, int PX>
void launch_t(int64_t channels, hipStream_t s, const void* y, const void* z, const float* gamma,
              const float* beta, float eps, void* out, int P, int64_t pixels) {
    constexpr int kGroups = kThreads / PX;
    const dim3 grid(static_cast<unsigned>((pixels + PX - 1) / PX));
    const T* yy = static_cast<const T*>(y);
    const T* zz = static_cast<const T*>(z);
    T* oo = static_cast<T*>(out);
    const int Dc = static_cast<int>(channels);
    const int64_t j = (channels + kGroups - 1) / kGroups;
    if (j <= 4)
        hipLaunchKernelGGL((k_out_norm<T, 4, PX>), grid, dim3(kThreads), 0, s, yy, zz, gamma, beta,
                           eps, oo, Dc, P, pixels);
    else if (j <= 8)
        hipLaunchKernelGGL((k_out_norm<T, 8, PX>), grid, dim3(kThreads), 0, s, yy, zz, gamma, beta,
                           eps, oo, Dc, P, pixels);
    else if (j <= 16)
        hipLaunchKernelGGL((k_out_norm<T, 16, PX>), grid, dim3(kThreads), 0, s, yy, zz, gamma, beta,
                           eps, oo, Dc, P, pixels);
    else if (j <= 32)
        hipLaunchKernelGGL((k_out_norm<T, 32, PX>), grid, dim3(kThreads), 0, s, yy, zz, gamma, beta,
                           eps, oo, Dc, P, pixels);
    else
        hipLaunchKernelGGL((k_out_norm<T, 0, PX>), grid, dim3(kThreads), 0, s, yy, zz, gamma, beta,
                           eps, oo, Dc, P, pixels);
}

}  // namespace

vmb_status launch_out_norm(const void* y, const void* z, const float* gamma, const float* beta,
                           float eps, void* out, int64_t batch, int64_t channels, int64_t P,
                           vmb_dtype dt, hipStream_t s) {
    const int64_t pixels = batch * P;
    if ((pixels + 3) / 4 > int64_t{0x7fffffff}) return VMB_ERR_UNSUPPORTED;
    const int v = dt == VMB_F32 ? vec_pixels<float>() : vec_pixels<bf16_t>();
    const int64_t vectors = batch * ((P + v - 1) / v);
    // vectors when the grid still covers the chip (below, the narrower tiles
    // of single pixels do: 32 x 14x14, 196 segments, 13 us either way)
    if (P >= v && channels <= kVecMaxJ * kVecGroups && vectors >= 8 * 256) {
        if (dt == VMB_F32)
            launch_vec<float>(s, y, z, gamma, beta, eps, out, int(channels), int(P), vectors);
        else
            launch_vec<bf16_t>(s, y, z, gamma, beta, eps, out, int(channels), int(P), vectors);
        return check_launch();
    }
    // widest tile (64-byte row segments) whose grid has 512 workgroups, as
    // long as every thread keeps at least four channels (the group sums are
    // added serially, so idle groups cost)
    auto shrink = [&](int px) {
        int k = 0;
        while (k < 2 && (pixels + px - 1) / px < 512 && channels >= 4 * (kThreads / (px / 2)))
            px /= 2, ++k;
        return px;
    };
    if (dt == VMB_F32) {
        const int px = shrink(16);
        if (px == 16) launch_t<float, 16>(channels, s, y, z, gamma, beta, eps, out, int(P), pixels);
        else if (px == 8) launch_t<float, 8>(channels, s, y, z, gamma, beta, eps, out, int(P), pixels);
        else launch_t<float, 4>(channels, s, y, z, gamma, beta, eps, out, int(P), pixels);
    } else {
        const int px = shrink(32);
        if (px == 32) launch_t<bf16_t, 32>(channels, s, y, z, gamma, beta, eps, out, int(P), pixels);
        else if (px == 16) launch_t<bf16_t, 16>(channels, s, y, z, gamma, beta, eps, out, int(P), pixels);
        else launch_t<bf16_t, 8>(channels, s, y, z, gamma, beta, eps, out, int(P), pixels);
    }
    return check_launch();
}

}  // namespace vmb
