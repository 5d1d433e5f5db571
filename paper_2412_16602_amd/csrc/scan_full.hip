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
// 4-byte boundary, so those shapes take the lane-per-channel kernel.
bool use_chunked_full(const ScanArgs& a) {
    return a.N == 16 && a.L > kShortMaxL && !(a.in_dt == VMB_BF16 && (a.L & 1));
}

vmb_status launch_full_scan(const ScanArgs& a) {
    // the zero-order-hold B runs in the tile, positions-over-lanes and lane
    // kernels (not the short-sequence one: those shapes take the tile kernel)
    const bool zoh = (a.options & VMB_SCAN_ZOH) != 0;
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
