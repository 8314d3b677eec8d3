// rows.hpp -- row-wise scan of the tile counts of a partition (sort.hip: by
// digit or flag; resolve.hip: by target range).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace abm {
namespace {

// Exclusive scan in place of row r = blockIdx.x of n_tiles counts (the tile
// counts of one radix digit, of the set flags, or of one target range); totals[r] = the row's sum.
// One workgroup of 1024 threads per row, four consecutive counts per thread
// (one round for up to 4096 tiles, i.e. 2^24 keys).
constexpr int kScanThreads = 1024;

__global__ __launch_bounds__(kScanThreads) void k_scan_rows(uint32_t* rows, uint32_t n_tiles,
                                                            uint32_t* totals) {
    uint32_t* counts = rows + int64_t(blockIdx.x) * n_tiles;
    __shared__ uint32_t wtot[kScanThreads / 64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint32_t carry = 0;
    for (uint32_t c0 = 0; c0 < n_tiles; c0 += 4 * kScanThreads) {
        const uint32_t i = c0 + 4 * threadIdx.x;
        uint32_t v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = i + q < n_tiles ? counts[i + q] : 0u;
        const uint32_t mine = v[0] + v[1] + v[2] + v[3];
        uint32_t x = mine;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t y = __shfl_up(x, o, 64);
            if (lane >= o) x += y;
        }
        if (lane == 63) wtot[w] = x;
        __syncthreads();
        uint32_t before = 0, all = 0;
#pragma unroll
        for (int q = 0; q < kScanThreads / 64; ++q) {
            before += q < w ? wtot[q] : 0u;
            all += wtot[q];
        }
        uint32_t ex = carry + before + x - mine;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (i + q < n_tiles) {
                counts[i + q] = ex;
                ex += v[q];
            }
        carry += all;
        __syncthreads();   // wtot is reused by the next round
    }
    if (threadIdx.x == 0) totals[blockIdx.x] = carry;
}

}  // namespace
}  // namespace abm
