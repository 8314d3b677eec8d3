// wave.hpp -- scans and reductions over the 64 lanes of a wave with DPP lane
// moves (register to register; a __shfl goes through the LDS and costs about
// ten times the latency), and the ordering point for data that lanes of one
// wave hand each other through LDS.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace abm {

// x of the lane `CTRL` moves from, or 0 where the move has no source or the
// lane's row is not in ROWS.
template <int CTRL, int ROWS = 0xF>
__device__ __forceinline__ int32_t dpp_move(int32_t x) {
    return __builtin_amdgcn_update_dpp(0, x, CTRL, ROWS, 0xF, false);
}

// Inclusive prefix sum over the wave.  row_shr 1, 2, 4, 8 scan each row of 16
// lanes; row_bcast 15 adds rows 0 and 2 into rows 1 and 3, row_bcast 31 the
// lower half into the upper.  All 64 lanes must be active.
__device__ __forceinline__ int32_t wave_incl_sum(int32_t x) {
    x += dpp_move<0x111>(x);
    x += dpp_move<0x112>(x);
    x += dpp_move<0x114>(x);
    x += dpp_move<0x118>(x);
    x += dpp_move<0x142, 0xA>(x);
    x += dpp_move<0x143, 0xC>(x);
    return x;
}

// Maximum over the wave of values >= 0, in every lane.  All lanes active.
__device__ __forceinline__ int32_t wave_max_nonneg(int32_t x) {
    x = max(x, dpp_move<0x111>(x));
    x = max(x, dpp_move<0x112>(x));
    x = max(x, dpp_move<0x114>(x));
    x = max(x, dpp_move<0x118>(x));
    x = max(x, dpp_move<0x142, 0xA>(x));
    x = max(x, dpp_move<0x143, 0xC>(x));
    return __builtin_amdgcn_readlane(x, 63);
}

// Orders the LDS accesses of this wave's lanes: what any lane wrote before is
// seen by every lane after.  (The LDS serves one wave's accesses in order; the
// fence keeps the compiler from moving them.)
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

}  // namespace abm
