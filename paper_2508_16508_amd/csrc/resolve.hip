// resolve.hip -- abm_resolve_conflicts: many claimants for one resource.
//
// The priority and the claim index are packed into one 64-bit key
// (prio << 32 | claim), so a single unsigned atomicMin per claim both picks the
// lowest priority and breaks ties by the lower index; the winner is then a
// plain equality test against the reduced key.  Three launches because each
// pass depends on the whole previous pass: reset, reduce, read back.
//
// Device-wide atomics run at a fixed rate (26 G a second, whatever their width
// or where they go; slower still on one address), which bounds the reduction.  With a workspace, many
// claims are therefore partitioned by target first, into at most 512 ranges of
// equal length whose keys fit one workgroup's LDS, and reduced there:
//   count    live claims per tile and range;
//   scan     the ranges' rows of tile counts;
//   move     each tile's claims, (target, key), to their ranges, staged in LDS
//            in range order so that runs are written;
//   reduce   one workgroup per range: atomicMin in LDS, then best, winner and
//            the winners' won[] (a range holding more claims than a chunk is cut
//            into chunks, merged by device-wide atomics);
//   finish   winner and won[] of the ranges that were cut.
// 2^22 claims on 2^20 targets: 14 + 4 + 25 + 21 + 4 us of kernels against 9 +
// 143 + 44.  The move is bound by the latency of its LDS rounds at 24 waves a
// CU, the reduction by that of one workgroup a range.
#include <hip/hip_runtime.h>

#include "abm.h"
#include "common.hpp"
#include "rows.hpp"
#include "scan.hpp"
#include "wave.hpp"

namespace abm {
namespace {

constexpr int kBlock = 256;

__global__ __launch_bounds__(kBlock) void k_reset_keys(uint64_t* __restrict__ best, int64_t n) {
    const int64_t i = int64_t(blockIdx.x) * kBlock + threadIdx.x;
    if (i < n) best[i] = ~0ull;
}

__device__ __forceinline__ bool claim_live(int64_t c, const int32_t* target, const uint8_t* active,
                                           int64_t n_targets, int32_t& t) {
    t = target[c];
    return (active == nullptr || active[c] != 0) && t >= 0 && int64_t(t) < n_targets;
}

__global__ __launch_bounds__(kBlock) void k_claim(const int32_t* __restrict__ target,
                                                  const uint32_t* __restrict__ prio,
                                                  const uint8_t* __restrict__ active,
                                                  int64_t n_claims, int64_t n_targets,
                                                  uint64_t* best) {
    const int64_t c = int64_t(blockIdx.x) * kBlock + threadIdx.x;
    if (c >= n_claims) return;
    int32_t t;
    if (!claim_live(c, target, active, n_targets, t)) return;
    const uint64_t key = (uint64_t(prio[c]) << 32) | uint32_t(c);
    atomicMin(reinterpret_cast<unsigned long long*>(best + t), static_cast<unsigned long long>(key));
}

// Threads [0, n_claims) fill won[], threads [0, n_targets) fill winner[].
__global__ __launch_bounds__(kBlock) void k_readback(const int32_t* __restrict__ target,
                                                     const uint32_t* __restrict__ prio,
                                                     const uint8_t* __restrict__ active,
                                                     int64_t n_claims, int64_t n_targets,
                                                     const uint64_t* __restrict__ best,
                                                     int32_t* __restrict__ winner,
                                                     uint8_t* __restrict__ won) {
    const int64_t i = int64_t(blockIdx.x) * kBlock + threadIdx.x;
    if (i < n_claims) {
        int32_t t;
        uint8_t w = 0;
        if (claim_live(i, target, active, n_targets, t)) {
            const uint64_t key = (uint64_t(prio[i]) << 32) | uint32_t(i);
            w = best[t] == key ? 1 : 0;
        }
        won[i] = w;
    }
    if (i < n_targets) {
        const uint64_t b = best[i];
        winner[i] = b == ~0ull ? -1 : int32_t(uint32_t(b));
    }
}

// ------------------------------------------------------------ by target range
constexpr int kRanges = 512;
constexpr int kMoveThreads = kRanges;             // a thread per range in the scans
constexpr int kMoveItems = 8;
constexpr int64_t kMoveTile = int64_t(kMoveThreads) * kMoveItems;   // 4096 claims
constexpr int kReduceThreads = 1024;
constexpr int kMaxSpanBits = 14;                  // 16384 keys: 128 KiB of LDS
constexpr uint32_t kXcds = 8;

struct RangeArgs {
    const int32_t* target;
    const uint32_t* prio;
    const uint8_t* active;
    int64_t n_claims, n_targets;
    uint64_t* best;
    int32_t* winner;
    uint8_t* won;
    uint32_t* counts;        // [kRanges][n_tiles]
    uint32_t* totals;        // [kRanges]
    int32_t* out_target;     // claims in range order
    uint64_t* out_key;
    uint32_t n_tiles;
    uint32_t shift;          // range = target >> shift
    uint32_t chunk;          // claims of one workgroup of the reduction
};

// The claims of this thread: bit k of the result is set when claim
// t * kMoveTile + k * kMoveThreads + thread is live; its target in tg[k].
__device__ __forceinline__ uint32_t load_claims(const RangeArgs& a, uint32_t t,
                                                int32_t (&tg)[kMoveItems]) {
    const int64_t c0 = int64_t(t) * kMoveTile + threadIdx.x;
    uint8_t on[kMoveItems];
#pragma unroll
    for (int k = 0; k < kMoveItems; ++k) {
        const int64_t c = c0 + k * kMoveThreads, at = c < a.n_claims ? c : a.n_claims - 1;
        tg[k] = a.target[at];
        on[k] = a.active ? a.active[at] : uint8_t(1);
    }
    uint32_t live = 0;
#pragma unroll
    for (int k = 0; k < kMoveItems; ++k)
        if (c0 + k * kMoveThreads < a.n_claims && on[k] != 0 && tg[k] >= 0 &&
            int64_t(tg[k]) < a.n_targets)
            live |= 1u << k;
    return live;
}

__global__ __launch_bounds__(kMoveThreads) void k_range_count(RangeArgs a) {
    __shared__ uint32_t hist[kRanges];
    const uint32_t t = blockIdx.x;
    int32_t tg[kMoveItems];
    const uint32_t live = load_claims(a, t, tg);
    hist[threadIdx.x] = 0;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kMoveItems; ++k)
        if ((live >> k) & 1u) atomicAdd(&hist[uint32_t(tg[k]) >> a.shift], 1u);
    for (int64_t i = int64_t(t) * kMoveThreads + threadIdx.x; i < a.n_targets;
         i += int64_t(gridDim.x) * kMoveThreads)
        a.best[i] = ~0ull;
    __syncthreads();
    a.counts[int64_t(threadIdx.x) * a.n_tiles + t] = hist[threadIdx.x];
}

// Exclusive prefix of one value per range; the block's threads are the ranges.
__device__ __forceinline__ uint32_t range_scan(uint32_t v, uint32_t* lds) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint32_t incl = uint32_t(wave_incl_sum(int32_t(v)));
    if (lane == 63) lds[w] = incl;
    __syncthreads();
    uint32_t before = incl - v;
    for (int q = 0; q < w; ++q) before += lds[q];
    __syncthreads();
    return before;
}

// (Consecutive tiles on one XCD: the ends of the runs they share meet in one
// L2.)
__global__ __launch_bounds__(kMoveThreads) void k_range_move(RangeArgs a) {
    __shared__ uint32_t cnt[kRanges], start[kRanges], lds[kMoveThreads / 64];
    __shared__ int64_t goff[kRanges];
    __shared__ int32_t s_target[kMoveTile];
    __shared__ uint64_t s_key[kMoveTile];
    const uint32_t t = (blockIdx.x % kXcds) * ((a.n_tiles + kXcds - 1) / kXcds) + blockIdx.x / kXcds;
    if (t >= a.n_tiles) return;
    int32_t tg[kMoveItems];
    uint32_t pr[kMoveItems], rank[kMoveItems];
    const uint32_t live = load_claims(a, t, tg);
    const int64_t c0 = int64_t(t) * kMoveTile + threadIdx.x;
#pragma unroll
    for (int k = 0; k < kMoveItems; ++k) {
        const int64_t c = c0 + k * kMoveThreads;
        pr[k] = a.prio[c < a.n_claims ? c : a.n_claims - 1];
        // (here and not in the count: won may be the array that active is, and
        // every claim counted has to be moved)
        if (c < a.n_claims) a.won[c] = 0;
    }
    const uint32_t before_tile = a.counts[int64_t(threadIdx.x) * a.n_tiles + t];
    const uint32_t total = a.totals[threadIdx.x];
    cnt[threadIdx.x] = 0;
    __syncthreads();
    // (the order within a range does not matter: the key holds the claim)
#pragma unroll
    for (int k = 0; k < kMoveItems; ++k)
        rank[k] = (live >> k) & 1u ? atomicAdd(&cnt[uint32_t(tg[k]) >> a.shift], 1u) : 0u;
    __syncthreads();
    const uint32_t mine = cnt[threadIdx.x];
    const uint32_t st = range_scan(mine, lds);
    start[threadIdx.x] = st;
    goff[threadIdx.x] = int64_t(range_scan(total, lds)) + before_tile - int64_t(st);
    if (threadIdx.x == kMoveThreads - 1) lds[0] = st + mine;
    __syncthreads();
    const uint32_t n = lds[0];
#pragma unroll
    for (int k = 0; k < kMoveItems; ++k)
        if ((live >> k) & 1u) {
            const uint32_t p = start[uint32_t(tg[k]) >> a.shift] + rank[k];
            s_target[p] = tg[k];
            s_key[p] = (uint64_t(pr[k]) << 32) | uint32_t(c0 + k * kMoveThreads);
        }
    __syncthreads();
    for (uint32_t p = threadIdx.x; p < n; p += kMoveThreads) {
        const int32_t x = s_target[p];
        const int64_t dst = goff[uint32_t(x) >> a.shift] + p;
        a.out_target[dst] = x;
        a.out_key[dst] = s_key[p];
    }
}

// Workgroup b of the reduction: its range, first and last claim, and whether
// the range is cut.  Every range has one workgroup at least.
__global__ __launch_bounds__(kReduceThreads) void k_range_reduce(RangeArgs a) {
    extern __shared__ uint64_t keys[];
    __shared__ uint32_t lds[kReduceThreads / 64];
    __shared__ uint32_t s_item[4];                // range, first, end, cut
    const bool range = threadIdx.x < kRanges;
    const uint32_t total = range ? a.totals[threadIdx.x] : 0u;
    const uint32_t parts = range ? (total > a.chunk ? (total + a.chunk - 1) / a.chunk : 1u) : 0u;
    const uint32_t first_item = range_scan(parts, lds), first_claim = range_scan(total, lds);
    if (threadIdx.x == 0) s_item[0] = kRanges;
    __syncthreads();
    const uint32_t b = blockIdx.x;
    if (b >= first_item && b < first_item + parts) {
        const uint32_t c = (b - first_item) * a.chunk;
        s_item[0] = threadIdx.x;
        s_item[1] = first_claim + c;
        s_item[2] = first_claim + (total - c < a.chunk ? total : c + a.chunk);
        s_item[3] = parts > 1;
    }
    const uint32_t span = 1u << a.shift;
    for (uint32_t i = threadIdx.x; i < span; i += kReduceThreads) keys[i] = ~0ull;
    __syncthreads();
    const uint32_t r = s_item[0], end = s_item[2];
    if (r >= kRanges) return;
    typedef __attribute__((address_space(3))) unsigned long long lds_u64;
    for (uint32_t c0 = s_item[1] + threadIdx.x; c0 < end; c0 += 4 * kReduceThreads) {
        int32_t x[4];
        uint64_t k[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t c = c0 + u * kReduceThreads, at = c < end ? c : end - 1;
            x[u] = a.out_target[at];
            k[u] = a.out_key[at];
        }
        // (past the end: the last claim once more, which changes nothing)
#pragma unroll
        for (int u = 0; u < 4; ++u)
            __hip_atomic_fetch_min((lds_u64*)&keys[uint32_t(x[u]) & (span - 1)],
                                   static_cast<unsigned long long>(k[u]), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    __syncthreads();
    const int64_t t0 = int64_t(r) << a.shift;
    const uint32_t here = a.n_targets - t0 < int64_t(span) ? uint32_t(max(a.n_targets - t0, int64_t(0))) : span;
    if (s_item[3]) {
        for (uint32_t i = threadIdx.x; i < here; i += kReduceThreads)
            if (keys[i] != ~0ull)
                atomicMin(reinterpret_cast<unsigned long long*>(a.best + t0 + i),
                          static_cast<unsigned long long>(keys[i]));
        return;
    }
    for (uint32_t i = threadIdx.x; i < here; i += kReduceThreads) {
        const uint64_t k = keys[i];
        a.best[t0 + i] = k;
        a.winner[t0 + i] = k == ~0ull ? -1 : int32_t(uint32_t(k));
        if (k != ~0ull) a.won[uint32_t(k)] = 1;
    }
}

// The ranges that were cut.
__global__ __launch_bounds__(kReduceThreads) void k_range_finish(RangeArgs a) {
    if (a.totals[blockIdx.x] <= a.chunk) return;
    const int64_t t0 = int64_t(blockIdx.x) << a.shift;
    for (int64_t i = t0 + threadIdx.x; i < t0 + (int64_t(1) << a.shift) && i < a.n_targets;
         i += kReduceThreads) {
        const uint64_t k = a.best[i];
        a.winner[i] = k == ~0ull ? -1 : int32_t(uint32_t(k));
        if (k != ~0ull) a.won[uint32_t(k)] = 1;
    }
}

// Claims from which the partition is worth its five launches.  With as many
// targets as claims, in us, atomics against ranges: 2^19 claims 38 and 44,
// 2^20 67 and 52, 2^22 229 and 97; with a quarter as many targets 33 and 42,
// 56 and 46, 199 and 75.  Past 16384 targets a range (2^23 in all) the keys of
// a range no longer fit the LDS.
constexpr int64_t kRangeClaims = int64_t(1) << 20;

// The shift of the target ranges, or -1 when the call is not partitioned.
int range_shift(int64_t n_claims, int64_t n_targets) {
    if (n_claims < kRangeClaims || n_targets < 1) return -1;
    int shift = 0;
    while (((n_targets - 1) >> shift) >= kRanges) ++shift;
    return shift <= kMaxSpanBits ? shift : -1;
}

int64_t range_tiles(int64_t n_claims) { return tiles_for(n_claims, kMoveTile); }
int64_t up256(int64_t b) { return (b + 255) / 256 * 256; }

size_t range_ws_bytes(int64_t n_claims) {
    return size_t(up256(4 * kRanges * range_tiles(n_claims)) + up256(4 * kRanges) +
                  up256(4 * n_claims) + up256(8 * n_claims));
}

int check_resolve(int64_t n_claims, const int32_t* target, const uint32_t* prio,
                  int64_t n_targets, const uint64_t* best, const int32_t* winner,
                  const uint8_t* won) {
    // winner[] holds claim indices as int32, with -1 for "no claim"
    if (n_claims < 0 || n_claims > kMaxIndex)
        return fail(ABM_E_INVALID, "n_claims must be in [0, 2^31)");
    if (n_targets < 0 || n_targets > kMaxIndex)
        return fail(ABM_E_INVALID, "n_targets must be in [0, 2^31)");
    if (n_claims > 0 && (!target || !prio || !won))
        return fail(ABM_E_INVALID, "target, prio or won is NULL");
    if (n_targets > 0 && (!best || !winner)) return fail(ABM_E_INVALID, "best or winner is NULL");
    return check_device();
}

}  // namespace
}  // namespace abm

using namespace abm;

extern "C" int abm_resolve_conflicts(int64_t n_claims, const int32_t* target, const uint32_t* prio,
                                     const uint8_t* active, int64_t n_targets, uint64_t* best,
                                     int32_t* winner, uint8_t* won, void* stream) {
    const int rc = check_resolve(n_claims, target, prio, n_targets, best, winner, won);
    if (rc != ABM_OK) return rc;
    hipStream_t st = as_stream(stream);
    if (n_targets > 0)
        hipLaunchKernelGGL(k_reset_keys, dim3(tiles_for(n_targets, kBlock)), dim3(kBlock), 0, st,
                           best, n_targets);
    if (n_claims > 0 && n_targets > 0)
        hipLaunchKernelGGL(k_claim, dim3(tiles_for(n_claims, kBlock)), dim3(kBlock), 0, st, target,
                           prio, active, n_claims, n_targets, best);
    const int64_t m = n_claims > n_targets ? n_claims : n_targets;
    if (m > 0)
        hipLaunchKernelGGL(k_readback, dim3(tiles_for(m, kBlock)), dim3(kBlock), 0, st, target,
                           prio, active, n_claims, n_targets, best, winner, won);
    return launch_status("resolve_conflicts");
}

extern "C" size_t abm_resolve_workspace_bytes(int64_t n_claims, int64_t n_targets) {
    if (n_claims < 0 || n_claims > kMaxIndex || n_targets < 0 || n_targets > kMaxIndex) return 0;
    return range_shift(n_claims, n_targets) < 0 ? 0 : range_ws_bytes(n_claims);
}

extern "C" int abm_resolve_conflicts_ws(int64_t n_claims, const int32_t* target,
                                        const uint32_t* prio, const uint8_t* active,
                                        int64_t n_targets, uint64_t* best, int32_t* winner,
                                        uint8_t* won, void* ws, size_t ws_bytes, void* stream) {
    const int shift = range_shift(n_claims, n_targets);
    if (shift < 0)
        return abm_resolve_conflicts(n_claims, target, prio, active, n_targets, best, winner, won,
                                     stream);
    const int rc = check_resolve(n_claims, target, prio, n_targets, best, winner, won);
    if (rc != ABM_OK) return rc;
    const size_t need = range_ws_bytes(n_claims);
    if (!ws || ws_bytes < need) {
        set_error("workspace has %zu bytes, needs %zu", ws_bytes, need);
        return ABM_E_WORKSPACE;
    }
    if ((reinterpret_cast<uintptr_t>(ws) & 255) != 0)
        return fail(ABM_E_WORKSPACE, "workspace must be 256-byte aligned");
    hipStream_t st = as_stream(stream);
    RangeArgs a;
    a.target = target;
    a.prio = prio;
    a.active = active;
    a.n_claims = n_claims;
    a.n_targets = n_targets;
    a.best = best;
    a.winner = winner;
    a.won = won;
    a.n_tiles = uint32_t(range_tiles(n_claims));
    a.shift = uint32_t(shift);
    // a chunk is twice an even share of the claims, so that ranges are cut where
    // targets crowd, but 65536 claims at most: few targets make few ranges, and
    // many claims make even ranges longer than one workgroup should walk alone
    // (2^26 claims on 2^20 targets, all ranges cut: 0.77 ms, 3.19 by atomics; 2^20
    // on 7: 0.10 and 4.19; on 2^20 targets, none cut, 2^22: 0.08 and 0.23)
    const int64_t ranges = ((n_targets - 1) >> shift) + 1;
    const int64_t share = 2 * ((n_claims + ranges - 1) / ranges);
    a.chunk = uint32_t(share < 16384 ? 16384 : (share > 65536 ? 65536 : share));
    char* p = static_cast<char*>(ws);
    a.counts = reinterpret_cast<uint32_t*>(p);
    p += up256(4 * kRanges * int64_t(a.n_tiles));
    a.totals = reinterpret_cast<uint32_t*>(p);
    p += up256(4 * kRanges);
    a.out_key = reinterpret_cast<uint64_t*>(p);
    p += up256(8 * n_claims);
    a.out_target = reinterpret_cast<int32_t*>(p);
    const uint32_t moves = (a.n_tiles + kXcds - 1) / kXcds * kXcds;
    const uint32_t parts = uint32_t(n_claims / a.chunk) + kRanges;   // an upper bound
    hipLaunchKernelGGL(k_range_count, dim3(a.n_tiles), dim3(kMoveThreads), 0, st, a);
    hipLaunchKernelGGL(k_scan_rows, dim3(kRanges), dim3(kScanThreads), 0, st, a.counts, a.n_tiles,
                       a.totals);
    hipLaunchKernelGGL(k_range_move, dim3(moves), dim3(kMoveThreads), 0, st, a);
    hipLaunchKernelGGL(k_range_reduce, dim3(parts), dim3(kReduceThreads), size_t(8) << shift, st, a);
    hipLaunchKernelGGL(k_range_finish, dim3(uint32_t(ranges)), dim3(kReduceThreads), 0, st, a);
    return launch_status("resolve_conflicts");
}
