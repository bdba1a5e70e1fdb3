// Dispatch of the matrix-core variants with element-aligned accesses (ANY), shared by the inference and the training unit.
//
// What is different from the plain variants: 16-byte accesses that assume no alignment; a last group of 8 columns of x that
// reaches past the row is read 8 columns from its end and moved into place in registers (columns past the end are zeros, and
// no other row's values come in); a lane's 32 bits of sign(A) are cut out of two words; the last group of 8 columns of y is
// computed 8 columns from the end and stores only the columns that no other group has; requests that a wave has no use for
// (chunks or blocks past its share) are not made, since with so little work per call they are a third of it.
//
// Every call that the plain variants decline comes here first, also pools of adapters with several envelopes at r > 16 or 32.
// Measured against the general kernel on 28 small shapes (17 to 1001 columns, 1 to 1024 rows, r = 1 to 8) it is 1.1 to 2.3 times
// as fast on each, beyond that 3 to 50 times (us, general kernel in brackets): 1500 x 1000 -> 3001, r = 12 8.5 (32.8); 4000 x 5001
// -> 5001, r = 16 36.4 (352); 16 x 999 -> 12777, r = 57 7.2 (136); 1 x 33 -> 17, r = 1 3.1 (3.7).  Bound: at 4000 rows of 5001 the
// streams (3.3 TB/s; rows that start inside a cache line share it with their neighbours), at a few rows the latency of the
// chain.
// Where the general kernel would still be faster: a batch of more than 512 rows at r <= 8 whose every row has another adapter (1500 x
// 1353 -> 140, r = 2 18.7 us against 12.3, 600 rows 10.2 against 9.0); sorted by adapter, as batches of that size are, the same calls
// take 7.7 and 6.0, and the host does not see the order.
//
// u is held as fp16 hi + lo, 22 bits of its row's largest entry, where the general kernel holds fp32: error against 64 bits on 40 odd
// shapes, with y_base and with y_base = 0, 1.0000 times the general kernel's (at most 1.000001).
#pragma once
#include "lordba_fwd_impl.h"

namespace {

// 8-row tiles on 8 waves throughout.  Few tiles split their output blocks as grid mode 2 does; otherwise one workgroup per tile.
template <int RB, int L>
lordba_status launch_any_depth(const FwdArgs& a, hipStream_t stream) {
    // chunks in flight per wave where they do not all fit: two where the accumulators of three or four envelopes leave no room for
    // more (with four chunks, up to 72 registers were spilled)
    constexpr int kDeep = RB * L >= 9 ? 2 : 4;
    const bool shallow = (a.d_in + 127) / 128 <= 2 * 8;  // every wave's chunks of d_in are in flight at once
    if (a.ids != nullptr) {
        return shallow ? launch_mfma_gm<RB, 8, 8, 2, true, 0, 4, L, true>(a, stream)
                       : launch_mfma_gm<RB, 8, 8, kDeep, false, 0, 4, L, true>(a, stream);
    }
    return shallow ? launch_mfma_gm<RB, 8, 8, 2, true, 0, 2, L, true>(a, stream)
                   : launch_mfma_gm<RB, 8, 8, kDeep, false, 0, 2, L, true>(a, stream);
}

template <int L>
lordba_status launch_any_rb(const FwdArgs& a, hipStream_t stream) {
    switch ((a.r + 15) / 16) {
        case 1: return launch_any_depth<1, L>(a, stream);
        case 2: return launch_any_depth<2, L>(a, stream);
        case 3: return launch_any_depth<3, L>(a, stream);
        default:
            if constexpr (L <= 3) return launch_any_depth<4, L>(a, stream);
            return LORDBA_ERR_ALGO;  // (the partial tiles of four envelopes need more than the 160 KiB of LDS)
    }
}

lordba_status launch_any(const FwdArgs& a, hipStream_t stream) {
    // a whole group of 8 columns on either side, and two words of sign(A)
    if (a.d_in < 8 || a.d_out < 8 || static_cast<int64_t>(a.r) * a.d_in <= 32) return LORDBA_ERR_ALGO;
    switch (a.ell) {
        case 1: return launch_any_rb<1>(a, stream);
        case 2: return launch_any_rb<2>(a, stream);
        case 3: return launch_any_rb<3>(a, stream);
        default: return launch_any_rb<4>(a, stream);
    }
}

}  // namespace
