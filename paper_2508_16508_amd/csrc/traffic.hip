// traffic.hip -- abm_traffic_init / abm_traffic_step: the three-lane traffic
// cellular automaton of Sec. 5.2 (Fig. 4), many roads at once (the paper
// vectorises it over roads with different car counts, Table 3).
//
// One workgroup owns one road for every step of a call, with a thread per cell:
// a thread keeps the slot of the car on its cell in a register.  Only the
// column before and the column after matter to a cell's step, so a step is one
// word per cell in LDS (its car and where that car wants to go), one workgroup
// barrier, and three words read back:
//   decide      a car in the exit column leaves under a green light and waits
//               under red; any other car picks left / straight / right
//               uniformly (a lane off the road means straight);
//   resolve     all claimants of a cell are cars of the column before it, so
//               the claimants and the cell work out the winner by themselves:
//               the cell, if free at the start of the step, admits the straight
//               arrival first, then the one from the lane below, then the one
//               from the lane above (the paper's priority mask);
//   move        winners move, losers wait, leaving cars are removed (alive =
//               0, stale fields kept);
//   spawn       every free entry cell whose draw is below T_spawn gets a car;
//               spawned cars take the lowest free slots in lane order.
// Draws are keyed on (seed + road, step, agent, purpose): lights and spawns per
// lane, lane changes per car slot.
#include <hip/hip_runtime.h>

#include "abm.h"
#include "common.hpp"
#include "rng.hpp"
#include "wave.hpp"

namespace abm {
namespace {

constexpr int kBlock = 256;        // threads of the clearing kernel
constexpr int kMaxLength = 1024;
constexpr int kMaxWaves = 16;
constexpr int32_t kNone = 3;       // a cell word with no car: target lane 3, slot 0

enum TrafficCol : int {
    kCars = 0, kExited, kMoved, kBlocked, kLost, kWaitingRed, kSpawned, kLaneChanges, kCols
};

struct TrafficArgs {
    int32_t L;
    uint32_t T_green, T_spawn, seed;
    int32_t *lane, *pos, *alive;
    int64_t* stats;       // [n_steps][n_roads][kCols] or null
    int32_t n_roads;
    uint32_t step0;
    int32_t n_steps;
};

// What one car slot became in this call.
enum SlotFate : uint8_t { kUntouched = 0, kLeftLane0 = 1, kSpawnedCar = 4 };   // 1-3: left from lane 0-2

// A cell's word: target lane of its car (kNone: it claims nothing) and the car
// slot + 1 above it (0: no car).
__device__ __forceinline__ int32_t word_slot(int32_t w) { return (w >> 2) - 1; }

// The lowest free slots of a road, ascending: `n` of them (at most kKeep),
// INT32_MAX above.  Uniform over the wave that keeps it.
struct LowSlots {
    static constexpr int kKeep = 6;
    int32_t f[kKeep], n;

    // Slot e is free now; `all` slots were free before it.  It joins when it is
    // among the lowest: below the last one kept, or if every free slot is kept.
    __device__ __forceinline__ void insert(int32_t e, int32_t all) {
        int32_t top = -1;
#pragma unroll
        for (int q = 0; q < kKeep; ++q) top = f[q] != INT32_MAX ? f[q] : top;
        if (n < all && e > top) return;
#pragma unroll
        for (int q = 0; q < kKeep; ++q) {
            const int32_t lo = min(f[q], e);
            e = max(f[q], e);
            f[q] = lo;
        }
        n = min(n + 1, int32_t(kKeep));
    }

    // The first c (0 to 3) are taken.
    __device__ __forceinline__ void drop(int32_t c) {
#pragma unroll
        for (int by = 1; by <= 2; by <<= 1) {
            const bool on = c & by;
#pragma unroll
            for (int q = 0; q < kKeep; ++q)
                f[q] = on ? (q + by < kKeep ? f[q + by] : INT32_MAX) : f[q];
        }
        n -= c;
    }

    // From the free bits of n slots.
    __device__ __forceinline__ void refill(const uint32_t* bits, int32_t slots) {
        const int lane = threadIdx.x & 63;
        uint64_t w = 0;                       // lane r: slots [64 r, 64 r + 64)
        if (lane * 64 < slots) w = (uint64_t(bits[2 * lane + 1]) << 32) | bits[2 * lane];
        n = 0;
#pragma unroll
        for (int q = 0; q < kKeep; ++q) {
            const uint64_t any = __ballot(w != 0);
            const int r = any ? __ffsll((unsigned long long)any) - 1 : 0;
            const int b = __ffsll((unsigned long long)w) - 1;          // of this lane's word
            const int32_t slot = r * 64 + __builtin_amdgcn_readlane(b, r);
            f[q] = any ? slot : INT32_MAX;
            n += any ? 1 : 0;
            if (lane == r) w &= w - 1;
        }
    }
};

// One step's statistics row from its waves' packed counts (cnt[0]: cars |
// moved << 16, cnt[1]: blocked | lane changes << 16) and ex: cars that left |
// waiting at red << 8 | spawned << 16.
__device__ __forceinline__ void write_row(const TrafficArgs& a, int32_t k,
                                          const uint32_t (*cnt)[kMaxWaves], int waves,
                                          uint32_t ex) {
    const int lane = threadIdx.x & 63;
    const uint32_t lo = uint32_t(wave_incl_sum(lane < waves ? int32_t(cnt[0][lane]) : 0));
    const uint32_t hi = uint32_t(wave_incl_sum(lane < waves ? int32_t(cnt[1][lane]) : 0));
    const uint32_t cm = uint32_t(__builtin_amdgcn_readlane(int32_t(lo), 63));
    const uint32_t bx = uint32_t(__builtin_amdgcn_readlane(int32_t(hi), 63));
    const int32_t exited = int32_t(ex & 0xFFu), red = int32_t((ex >> 8) & 0xFFu);
    const int32_t cars = int32_t(cm & 0xFFFFu), moved = int32_t(cm >> 16);
    const int32_t blocked = int32_t(bx & 0xFFFFu), changes = int32_t(bx >> 16);
    int32_t col = lane, v = cars;
    asm volatile("" : "+v"(col));   // (compared here, not held as eight masks all step)
    v = col == kExited ? exited : v;
    v = col == kMoved ? moved : v;
    v = col == kBlocked ? blocked : v;
    v = col == kLost ? cars - exited - red - blocked - moved : v;
    v = col == kWaitingRed ? red : v;
    v = col == kSpawned ? int32_t(ex >> 16) : v;
    v = col == kLaneChanges ? changes : v;
    if (lane < kCols) a.stats[(int64_t(k) * a.n_roads + blockIdx.x) * kCols + lane] = v;
}

// LDS per road of L columns: the words of two alternating steps, each five
// rows (the three lanes between two rows with no cars) of L + 2 columns (an
// empty one on either side), the free slots' bits and each slot's fate.
__host__ __device__ __forceinline__ int32_t grid_words(int32_t L) { return 5 * (L + 2); }
__host__ __device__ __forceinline__ int32_t free_words(int32_t L) { return (3 * L + 63) / 64 * 2; }

// A road on which cars share cells, as a caller may have placed them (no step
// puts a car on an occupied cell): such cars draw, claim and leave each for
// itself.  A thread per car slot, the slots in global memory; the LDS (6 bytes a
// slot) holds the lowest key that claims a cell, (direction priority << 24 |
// slot), whether a cell is occupied, and each car's target lane.
__device__ __forceinline__ void run_shared_cells(const TrafficArgs& a, int32_t* lds) {
    __shared__ uint32_t cnt[kCols], s_entry;
    const int32_t L = a.L, n = 3 * L, block = int32_t(blockDim.x);
    uint32_t* const claim = reinterpret_cast<uint32_t*>(lds);
    uint8_t* const occ = reinterpret_cast<uint8_t*>(claim + n);
    int8_t* const to = reinterpret_cast<int8_t*>(occ + n);
    const int64_t base = int64_t(blockIdx.x) * n;
    int32_t *const lane = a.lane + base, *const pos = a.pos + base, *const alive = a.alive + base;
    const int tid = threadIdx.x;
    const auto cell_of = [&](int32_t i) {     // -1: no car, or none of the road's
        const int32_t l = lane[i], x = pos[i];
        return alive[i] && l >= 0 && l < 3 && x >= 0 && x < L ? l * L + x : -1;
    };
    const auto key_of = [](int32_t from, int32_t lane_to, int32_t i) {
        return (lane_to == from ? 0u : (from < lane_to ? 1u : 2u)) << 24 | uint32_t(i);
    };
    for (int32_t k = 0; k < a.n_steps; ++k) {
        const uint64_t skey = stream_key(a.seed + blockIdx.x, a.step0 + uint32_t(k));
        __syncthreads();
        for (int32_t i = tid; i < n; i += block) {
            claim[i] = ~0u;
            occ[i] = 0;
        }
        if (tid < kCols) cnt[tid] = 0;
        if (tid == 0) s_entry = 0;
        __syncthreads();
        for (int32_t i = tid; i < n; i += block) {
            const int32_t c = cell_of(i);
            if (c >= 0) occ[c] = 1;
        }
        __syncthreads();
        for (int32_t i = tid; i < n; i += block) {
            const int32_t c = cell_of(i);
            if (c < 0) continue;
            atomicAdd(&cnt[kCars], 1u);
            const int32_t l = lane[i];
            to[i] = kNone;
            if (c - l * L == L - 1) continue;
            const int32_t nl = l + int32_t(scale(draw(skey, uint32_t(i), kTrafficLane), 3u)) - 1;
            const int32_t t = uint32_t(nl) > 2u ? l : nl, ahead = t * L + (c - l * L) + 1;
            if (occ[ahead]) {
                atomicAdd(&cnt[kBlocked], 1u);
            } else {
                to[i] = int8_t(t);
                atomicMin(&claim[ahead], key_of(l, t, i));
            }
        }
        __syncthreads();
        for (int32_t i = tid; i < n; i += block) {
            const int32_t c = cell_of(i);
            if (c < 0) continue;
            const int32_t l = lane[i], x = c - l * L, t = to[i];
            if (x == L - 1) {
                const bool green = draw(skey, uint32_t(l), kTrafficLight) < a.T_green;
                atomicAdd(&cnt[green ? kExited : kWaitingRed], 1u);
                if (green) alive[i] = 0;
                continue;
            }
            const bool moves = t != kNone && claim[t * L + x + 1] == key_of(l, t, i);
            if (moves) {
                atomicAdd(&cnt[kMoved], 1u);
                if (t != l) atomicAdd(&cnt[kLaneChanges], 1u);
                lane[i] = t;
                pos[i] = x + 1;
            } else {
                if (t != kNone) atomicAdd(&cnt[kLost], 1u);
                if (x == 0) atomicOr(&s_entry, 1u << l);
            }
        }
        __syncthreads();
        if (tid < 64) {
            const bool want = tid < 3 && !((s_entry >> tid) & 1u) &&
                              draw(skey, uint32_t(tid), kTrafficSpawn) < a.T_spawn;
            uint64_t left = __ballot(want);   // lanes still without a slot
            for (int32_t i0 = 0; i0 < n && left; i0 += 64) {
                uint64_t f = __ballot(i0 + tid < n && alive[i0 + tid] == 0);
                for (; f && left; f &= f - 1, left &= left - 1) {
                    const int32_t i = i0 + __ffsll((unsigned long long)f) - 1;
                    if (tid != 0) continue;
                    lane[i] = __ffsll((unsigned long long)left) - 1;
                    pos[i] = 0;
                    alive[i] = 1;
                    ++cnt[kSpawned];
                }
            }
        }
        __syncthreads();
        if (a.stats && tid < kCols)
            a.stats[(int64_t(k) * a.n_roads + blockIdx.x) * kCols + tid] = cnt[tid];
    }
}

// Wave 0 holds the entry and the exit column (lane l and lane 3 + l: lane l of
// the road) and spawns; the last wave holds no cell, draws what depends on no
// car for the steps to come and writes the statistics; the waves between them
// hold the other cells, R per thread (R = 1 up to 300 columns, 2 up to 599,
// else 4: at most 16 waves).
//
// What bounds a step: the instructions of its longest wave, one after the
// other (a wave alone on its SIMD takes 6 to 10 cycles for each); no bytes
// move but 64 of statistics.  So a thread has one cell and one draw, and the
// wave that spawns has few cells and keeps the lowest free slots at hand (a
// search of the free bits for three of them took 800 of a step's 3400 cycles).
// 500 roads of 3 x 100 cells, 1000 steps: 0.97 ms; with car slots and occupancy
// maps in LDS, LDS atomics and three barriers a step it was 1.95 ms, with a
// thread per column (three draws each) 1.53 ms.
template <int R>
__global__ __launch_bounds__(64 * kMaxWaves) void k_traffic_run(TrafficArgs a) {
    extern __shared__ int32_t grid[];
    __shared__ uint32_t s_cnt[2][2][kMaxWaves];   // packed counts of each wave
    __shared__ uint32_t s_ex[2];                  // left | waiting at red << 8 | spawned << 16
    __shared__ int32_t s_unplaced;                // cars without a cell of their own
    __shared__ uint4 s_pre[2];                    // a step's stream key (x, y), its lights and entry draws (z)
    const int32_t L = a.L, n = 3 * L, stride = L + 2, words = grid_words(L);
    uint32_t* const free_bits = reinterpret_cast<uint32_t*>(grid + 2 * words);
    uint8_t* const fate = reinterpret_cast<uint8_t*>(free_bits + free_words(L));
    const int64_t base = int64_t(blockIdx.x) * n;
    const uint32_t seed = a.seed + blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int waves = int(blockDim.x >> 6);

    // a step's key and the draws that depend on no car: bit l of the word, the
    // light of lane l; bit 3 + l, its entry draw.  Made two steps ahead by the last
    // wave
    const int helper = waves - 1;
    auto prepare_step = [&](int32_t step_k) {
        const uint64_t key = stream_key(seed, a.step0 + uint32_t(step_k));
        const bool light = lane < 3;
        const uint32_t d = draw(key, uint32_t(light ? lane : lane - 3), light ? kTrafficLight : kTrafficSpawn);
        const uint64_t hits = __ballot(lane < 6 && d < (light ? a.T_green : a.T_spawn));
        if (lane == 0)
            s_pre[step_k & 1] = uint4{uint32_t(key), uint32_t(key >> 32), uint32_t(hits), 0u};
    };
    // ---- load the road: car slots into the cells' words of step 0.  (A thread has
    // R slots at most, read together before the words are cleared)
    int32_t in_lane[R], in_pos[R], in_alive[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int32_t i = tid + r * int32_t(blockDim.x);
        in_lane[r] = i < n ? a.lane[base + i] : 0;
        in_pos[r] = i < n ? a.pos[base + i] : 0;
        in_alive[r] = i < n ? a.alive[base + i] : 1;
    }
    const int32_t sets = a.n_steps > 1 ? 2 : 1;
    for (int32_t i = tid; i < sets * words; i += int32_t(blockDim.x)) grid[i] = kNone;
    for (int32_t i = tid; i < n; i += int32_t(blockDim.x)) fate[i] = kUntouched;
    if (wave == helper) {
        prepare_step(0);
        if (a.n_steps > 1) prepare_step(1);
    }
    if (tid == 0) s_unplaced = 0;
    __syncthreads();
    int32_t cars = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int32_t i0 = wave * 64 + r * int32_t(blockDim.x), i = i0 + lane;
        const int32_t l = in_lane[r], x = in_pos[r];
        if (i < n && in_alive[r] && l >= 0 && l < 3 && x >= 0 && x < L) {
            grid[(l + 1) * stride + x + 1] = ((i + 1) << 2) | kNone;
            ++cars;
        }
        const uint64_t f = __ballot(in_alive[r] == 0);
        if (lane < 2 && i0 < n) free_bits[(i0 >> 5) + lane] = uint32_t(f >> (32 * lane));
    }
    __syncthreads();
    // wave 0 keeps the number of the free slots and the lowest of them
    int32_t n_free = 0;
    LowSlots low = {};
    if (wave == 0) {
        const int32_t words = free_words(L) / 2;
        const int32_t here = lane < words ? __popc(free_bits[2 * lane]) + __popc(free_bits[2 * lane + 1]) : 0;
        n_free = __builtin_amdgcn_readlane(wave_incl_sum(here), 63);
        low.refill(free_bits, n);
    }
    int32_t sl[R], cell[R], row[R], col[R];       // car slot (-1: none), cell's word index, lane, column
#pragma unroll
    for (int r = 0; r < R; ++r) {
        int32_t i = wave ? (tid - 64) + r * (int32_t(blockDim.x) - 128) : lane + r * 64;
        const int32_t len = L - 2;                // columns between the entry and the exit
        const bool ok = wave != helper && i < (wave ? 3 * len : 6);
        i = ok ? i : 0;
        row[r] = !ok ? 0 : (wave ? i / len : i % 3);
        col[r] = !ok ? -1 : (wave ? i % len + 1 : (i < 3 ? 0 : L - 1));
        cell[r] = ok ? (row[r] + 1) * stride + col[r] + 1 : 0;   // (word 0: never a car's)
        sl[r] = word_slot(grid[cell[r]]);
        cars -= sl[r] >= 0 ? 1 : 0;
    }
    cars = wave_incl_sum(cars);
    if (lane == 63 && cars) atomicAdd(&s_unplaced, cars);
    __syncthreads();
    if (s_unplaced != 0) {
        run_shared_cells(a, grid);
        return;
    }

    if (wave == 0) __builtin_amdgcn_s_setprio(3);   // every step waits for this wave
    for (int32_t k = 0; k < a.n_steps; ++k) {
        const int par = k & 1;
        int32_t* const now = grid + par * words;
        const uint4 pre = s_pre[par];
        const uint64_t skey = (uint64_t(pre.y) << 32) | pre.x;
        // ---- decide
        int32_t to[R];
#pragma unroll
        for (int r = 0; r < R && wave != helper; ++r) {
            const uint32_t d = draw(skey, uint32_t(sl[r]), kTrafficLane);
            const int32_t nl = row[r] + int32_t(scale(d, 3u)) - 1;
            int32_t t = uint32_t(nl) > 2u ? row[r] : nl;
            t = sl[r] < 0 || (wave == 0 && lane >= 3) ? kNone : t;
            to[r] = t;
            if (cell[r] > 0) now[cell[r]] = ((sl[r] + 1) << 2) | t;
        }
        // wave 0, while the others draw: the slots of the cars that leave are free
        bool leaves = false;                      // (this lane's car)
        int32_t want = 0, left = 0, waiting = 0;  // bits 0-2: entry draws, cars that leave, at red
        if (wave == 0) {
            const int32_t hits = __builtin_amdgcn_readfirstlane(int32_t(pre.z));
            const int32_t at_exit = int32_t(__ballot(lane >= 3 && lane < 6 && sl[0] >= 0)) >> 3;
            want = hits >> 3;
            left = at_exit & hits;
            waiting = at_exit & ~hits;
            if (lane >= 3 && lane < 6 && ((left >> (lane - 3)) & 1)) {
                leaves = true;
                atomicOr(&free_bits[sl[0] >> 5], 1u << (sl[0] & 31));
                fate[sl[0]] = uint8_t(kLeftLane0 + lane - 3);
            }
#pragma unroll
            for (int l = 0; l < 3; ++l)
                if ((left >> l) & 1) low.insert(__builtin_amdgcn_readlane(sl[0], 3 + l), n_free++);
        }
        __syncthreads();
        // ---- resolve and move.  A car reads the cell ahead and the cars of its
        // column that come first there; an empty cell reads the three cells it
        // can be entered from, in the order of its priorities
        uint32_t count = 0, count2 = 0;   // cars | moved << 16, blocked | changes << 16
#pragma unroll
        for (int r = 0; r < R && wave != helper; ++r) {
            const int32_t c = cell[r], t = to[r];
            const bool drives = t != kNone;
            const int32_t at = (t + 1) * stride + col[r] + 1;             // cell `to` of this column
            const int32_t i0 = drives ? at + 1 : (c > 0 ? c - 1 : 0);
            const int32_t i1 = drives ? at : (c > 0 ? c - 1 - stride : 0);
            const int32_t i2 = drives ? at - stride : (c > 0 ? c - 1 + stride : 0);
            const int32_t w0 = now[i0], w1 = now[i1], w2 = now[i2];
            const int32_t mine = drives ? t : row[r];
            const bool m0 = (w0 & 3) == mine, m1 = (w1 & 3) == mine, m2 = (w2 & 3) == mine;
            const bool blocked = drives && w0 >= 4;
            const bool moved = drives && !blocked &&
                               (t == row[r] || (!m1 && (t > row[r] || !m2)));
            const int32_t in = m0 ? w0 : (m1 ? w1 : (m2 ? w2 : kNone));
            const bool car = sl[r] >= 0;
            const bool waits = car && !moved && !(r == 0 && leaves);
            const bool on = c > 0;
            if (a.stats) {
                const uint64_t bc = __ballot(on && car), bm = __ballot(moved);
                const uint64_t bb = __ballot(blocked), bx = __ballot(moved && t != row[r]);
                count += uint32_t(__popcll(bc)) | uint32_t(__popcll(bm)) << 16;
                count2 += uint32_t(__popcll(bb)) | uint32_t(__popcll(bx)) << 16;
            }
            sl[r] = waits ? sl[r] : (car || !on ? -1 : word_slot(in));
        }
        if (a.stats && lane == 0) {
            s_cnt[par][0][wave] = count;
            s_cnt[par][1][wave] = count2;
        }
        // ---- spawn: the r-th spawning lane takes the r-th lowest free slot
        if (wave == 0) {
            const int32_t room = int32_t(__ballot(lane < 3 && sl[0] < 0)) & want;
            const int32_t asked = __popc(room);
            const int32_t spawned = asked < low.n ? asked : low.n;
            const int32_t mine = __popc(room & ((1 << (lane & 3)) - 1));
            if (lane < 3 && ((room >> lane) & 1) && mine < spawned) {
                sl[0] = mine == 0 ? low.f[0] : (mine == 1 ? low.f[1] : low.f[2]);
                fate[sl[0]] = kSpawnedCar;
                atomicAnd(&free_bits[sl[0] >> 5], ~(1u << (sl[0] & 31)));
            }
            low.drop(spawned);
            n_free -= spawned;
            if (low.n < 3 && low.n < n_free) {
                wave_lds_sync();
                low.refill(free_bits, n);
            }
            if (lane == 0)
                s_ex[par] = uint32_t(__popc(left)) | uint32_t(__popc(waiting)) << 8 |
                            uint32_t(spawned) << 16;
        }
        // (two steps ahead: its place was last read before this step's barrier)
        if (wave == helper && k + 2 < a.n_steps) prepare_step(k + 2);
        // the statistics of the step before (its counts are complete)
        if (a.stats && wave == helper && k > 0)
            write_row(a, k - 1, s_cnt[par ^ 1], waves, s_ex[par ^ 1]);
    }
    __syncthreads();
    if (a.stats && wave == helper && a.n_steps > 0)
        write_row(a, a.n_steps - 1, s_cnt[(a.n_steps - 1) & 1], waves, s_ex[(a.n_steps - 1) & 1]);
    // ---- write the road back: the cars from their cells, then the slots whose
    // car left (those keep the cell they left from)
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (sl[r] >= 0) {
            a.lane[base + sl[r]] = row[r];
            a.pos[base + sl[r]] = col[r];
            if (fate[sl[r]] == kSpawnedCar) a.alive[base + sl[r]] = 1;
        }
    for (int32_t i = tid; i < n; i += int32_t(blockDim.x)) {
        const int f = fate[i];
        if (f >= kLeftLane0 && f < kSpawnedCar) {
            a.lane[base + i] = f - kLeftLane0;
            a.pos[base + i] = L - 1;
            a.alive[base + i] = 0;
        }
    }
}

__global__ __launch_bounds__(kBlock) void k_traffic_clear(int32_t* lane, int32_t* pos,
                                                         int32_t* alive, int64_t n) {
    for (int64_t i = int64_t(blockIdx.x) * kBlock + threadIdx.x; i < n;
         i += int64_t(gridDim.x) * kBlock) {
        lane[i] = 0;
        pos[i] = 0;
        alive[i] = 0;
    }
}

int check_traffic(const abm_traffic_params* p, const abm_traffic_state* s) {
    if (!p || !s) return fail(ABM_E_INVALID, "params or state is NULL");
    if (p->length < 2 || p->length > kMaxLength)
        return fail(ABM_E_INVALID, "length must be in [2, 1024]");
    if (s->n_roads < 1 || s->n_roads > (1 << 20))
        return fail(ABM_E_INVALID, "n_roads must be in [1, 2^20]");
    if (!s->lane || !s->pos || !s->alive) return fail(ABM_E_INVALID, "car array is NULL");
    return ABM_OK;
}

}  // namespace
}  // namespace abm

using namespace abm;

extern "C" int abm_traffic_init(const abm_traffic_params* p, abm_traffic_state* s, void* stream) {
    int rc = check_traffic(p, s);
    if (rc != ABM_OK) return rc;
    rc = check_device();
    if (rc != ABM_OK) return rc;
    const int64_t n = int64_t(s->n_roads) * 3 * p->length;
    const int64_t blocks = tiles_for(n, kBlock) < 4096 ? tiles_for(n, kBlock) : 4096;
    hipLaunchKernelGGL(k_traffic_clear, dim3(uint32_t(blocks)), dim3(kBlock), 0, as_stream(stream),
                       s->lane, s->pos, s->alive, n);
    rc = launch_status("traffic_init");
    if (rc == ABM_OK) s->step = 0;
    return rc;
}

extern "C" int abm_traffic_step(const abm_traffic_params* p, abm_traffic_state* s,
                                int32_t n_steps, void* stream) {
    int rc = check_traffic(p, s);
    if (rc != ABM_OK) return rc;
    if (n_steps < 0) return fail(ABM_E_INVALID, "n_steps must be >= 0");
    rc = check_device();
    if (rc != ABM_OK) return rc;
    if (n_steps == 0) return ABM_OK;
    TrafficArgs a;
    a.L = p->length;
    a.T_green = p->T_green;
    a.T_spawn = p->T_spawn;
    a.seed = p->seed;
    a.lane = s->lane;
    a.pos = s->pos;
    a.alive = s->alive;
    a.stats = s->stats;
    a.n_roads = s->n_roads;
    a.step0 = s->step;
    a.n_steps = n_steps;
    const int32_t cells = 3 * (p->length - 2);   // between the entry and the exit column
    const int R = cells <= 64 * (kMaxWaves - 2) ? 1 : (cells <= 128 * (kMaxWaves - 2) ? 2 : 4);
    // (a thread's R slots cover the 3 length ones: the block holds cells / R threads
    // and two waves more)
    const size_t lds = size_t(8) * grid_words(p->length) + size_t(4) * free_words(p->length) +
                       size_t(3) * p->length;
    const dim3 grid(uint32_t(s->n_roads));
    const dim3 block(uint32_t(128 + (cells + 64 * R - 1) / (64 * R) * 64));
    hipStream_t st = as_stream(stream);
    if (R == 1)
        hipLaunchKernelGGL(k_traffic_run<1>, grid, block, lds, st, a);
    else if (R == 2)
        hipLaunchKernelGGL(k_traffic_run<2>, grid, block, lds, st, a);
    else
        hipLaunchKernelGGL(k_traffic_run<4>, grid, block, lds, st, a);
    rc = launch_status("traffic_step");
    if (rc == ABM_OK) s->step += uint32_t(n_steps);
    return rc;
}
