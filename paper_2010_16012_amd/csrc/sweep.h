// Work units of the degree-binned sweeps, shared by the pull and push
// kernels: every bin owns a contiguous range of work units, heaviest bin
// first (units run bin 5, 4, ..., 0); and the wavefront scans of the sweeps.
#pragma once

#include "pp_common.h"

namespace pp {

struct SweepPlan {
    int32_t block_off[PP_NUM_BINS + 1];
    int32_t list_off[PP_NUM_BINS + 1];
};

static SweepPlan sweep_plan(const BinPlan& p) {
    SweepPlan s;
    for (int b = 0; b <= PP_NUM_BINS; ++b) {
        s.block_off[b] = p.block_off[b];
        s.list_off[b] = p.list_off[b];
    }
    return s;
}

// Which bin does work unit `blk` belong to?  Units run bin 5, 4, ..., 0.
__device__ __forceinline__ int unit_bin(const SweepPlan& sp, int32_t blk) {
    int b = PP_NUM_BINS - 1;
#pragma unroll
    for (int i = PP_NUM_BINS - 1; i > 0; --i)
        if (blk >= sp.block_off[i - 1]) b = i - 1;
    return b;
}

// loads in flight per lane for a group of G lanes
template <int G>
constexpr int unroll_for() {
    return G >= 64 ? 8 : 4;
}

// Cross-lane moves through DPP: the data moves within the VALU, with no LDS
// round trip (the shuffles they replace were the tiled sweep's critical
// path).  A lane whose source lane lies outside its row, or whose row is
// masked off, gets 0.  Controls: row_shr:n = 0x110 + n; row_bcast:15 = 0x142
// (lane 15 of each row to the next row; rows 1 and 3 written); row_bcast:31
// = 0x143 (lane 31 to rows 2 and 3); wave_shr:1 = 0x138.
template <int CTRL, int ROWS = 0xf>
__device__ __forceinline__ int dpp_take(int x) {
    return __builtin_amdgcn_update_dpp(0, x, CTRL, ROWS, 0xf, false);
}
template <int CTRL, int ROWS = 0xf>
__device__ __forceinline__ float dpp_takef(float x) {
    return __int_as_float(dpp_take<CTRL, ROWS>(__float_as_int(x)));
}

// Inclusive prefix sum over the wavefront (all lanes active).
__device__ __forceinline__ int wave_incl_sum(int x) {
    x += dpp_take<0x111>(x);
    x += dpp_take<0x112>(x);
    x += dpp_take<0x114>(x);
    x += dpp_take<0x118>(x);
    x += dpp_take<0x142, 0xa>(x);
    x += dpp_take<0x143, 0xc>(x);
    return x;
}

// One step of an inclusive segmented scan: a lane that has not started a
// segment since the source lane adds the source's sum in front of its own.
template <int CTRL, int ROWS = 0xf>
__device__ __forceinline__ void seg_step(float& x, int& fresh) {
    const float xs = dpp_takef<CTRL, ROWS>(x);
    const int fs = dpp_take<CTRL, ROWS>(fresh);
    if (!fresh) {
        x = xs + x;
        fresh = fs;
    }
}

}  // namespace pp
