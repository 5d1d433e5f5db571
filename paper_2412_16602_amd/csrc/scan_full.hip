// scan_full.hip -- full (per-channel) selective scan: which kernel runs.
//
// Appendix A: eq. 3 recurrence h_t = Abar h_{t-1} + Bbar u_t, y_t = C h_t + D u_t,
// with Abar = exp(Delta A) (eq. 4, first line), Bbar u_t = Delta B_t u_t and
// Delta = softplus(delta + dt_bias) (eq. 6). One independent recurrence per
// (batch, direction k, channel d, state n); c = k*channels + d.
// exp(Delta*A) is evaluated as exp2((Delta*log2 e) * A) so the log2 e scaling
// is paid once per (channel, position), not once per state.
#include "vmb_internal.h"

namespace vmb {

// The chunked kernel copies B and C rows into LDS in pieces of 4 or 16
// bytes; a bf16 row of odd length has neither its start nor its end on a
// 4-byte boundary.
bool use_chunked_full(const ScanArgs& a) {
    return a.N == 16 && a.L > kShortMaxL && !(a.in_dt == VMB_BF16 && (a.L & 1));
}

// bf16, N = 16: with enough rows to fill the chip but too few for the tile
// kernel's 64-channel workgroups to, one wave per sequence is the fastest, since
// its loads and stores are whole vectors where the chunked kernel's are single
// elements. Measured (us, 2-D; chunked, short or tile kernel against rows):
// 56x56, 192 channels: 768 rows 40 / 60, 1536 73 / 70, 6144 273 / 150, 24576
// 765 / 531, 36864 928 / 785, 49152 1008 / 1039; 28x28: 1536 rows 40 / 22, 24576
// 218 / 170; 14x14: 3072 rows 29 / 16; 7x7 (L = 49): 6144 rows 22 / 23. (fp32,
// 56x56: 3072 rows 86 / 91, 12288 316 / 338: chunked.) Planes beyond 6144
// positions, for which the workspace has no column-major copies and both
// gather directions 1 and 3: 96x96, 24576 rows 3094 / 1526; 97x101, 17600 rows
// 11800 / 1424; 128x64, 16384 rows 2040 / 945.
// Rows that the tile kernel does not take (odd lengths) have no upper limit
// (short kernel: 15x15, 98304 rows 333 / 149; 7x13, 196608 rows 324 / 158), and
// above kShortMaxL none of the others takes them at all.
bool use_rows_full(const ScanArgs& a) {
    const int64_t rows = a.batch * a.K * a.channels;
    return a.N == 16 && a.in_dt == VMB_BF16 && a.L > 64 && rows >= 1200 &&
           (rows < 49152 || !tiles_take(a)) && a.batch <= 65535 && a.K <= 65535;
}

vmb_status launch_full_scan(const ScanArgs& a) {
    // the zero-order-hold B runs in the tile, positions-over-lanes and
    // one-wave-per-sequence kernels (not the short-sequence one: those shapes
    // take the tile kernel)
    const bool zoh = (a.options & VMB_SCAN_ZOH) != 0;
    if (!zoh && use_rows_full(a)) return launch_full_rows(a);
    const bool tiles =
        use_tiles_full(a) || (zoh && !use_chunked_full(a) && tiles_take(a));
    if (tiles || use_chunked_full(a) || (!zoh && use_short_full(a))) {
        auto run = [&](void* y_seq, const void* xt) {
            if (tiles) return launch_full_tiles(a, y_seq, xt);
            return use_short_full(a) ? launch_full_short(a, y_seq) : launch_full_chunked(a, y_seq, xt);
        };
        if (a.layout == VMB_LAYOUT_SEQ) return run(a.y, nullptr);
        // 2-D: the tile path, and the positions-over-lanes path on sequences of
        // several chunks, read directions 1 and 3 from column-major plane
        // copies in the workspace
        const void* xt = nullptr;
        const bool chunked_long = !tiles && !use_short_full(a) && a.L > kChunkedOneChunkMaxL;
        if ((tiles || chunked_long) && full_ws_has_xt(a.batch, a.K, a.channels, a.L, a.N)) {
            void* xtw = static_cast<char*>(a.ws) + full_ws_xt_offset(a.batch, a.K, a.channels, a.L);
            vmb_status st = launch_transpose_planes(a.u, xtw, a.batch, a.channels, a.H, a.W,
                                                    a.in_dt, a.stream);
            if (st != VMB_OK) return st;
            xt = xtw;
        }
        vmb_status st = run(a.ws, xt);
        if (st != VMB_OK) return st;
        return launch_cross_merge(a.ws, a.y, a.batch, a.channels, a.H, a.W, VMB_F32, a.out_dt,
                                  a.stream);
    }
    return launch_full_rows(a);
}

}  // namespace vmb
