// onchip.hpp -- a whole predation model advanced inside one workgroup's LDS.
//
// A model of up to 256 x 256 cells whose live agents lie in the lowest slots
// (children take the lowest free slots) fits the 160 KiB of one CU: four
// occupancy bits and one regrowth byte per cell, and 16 bits of position and
// the energy per slot.  The steps of a launch then touch no global memory;
// the state is read once at the start and written back once at the end.
//
// Why occupancy bits instead of claim words.  A cell's winners (the sheep that
// eats the grass, the sheep that is eaten, the wolf that eats) need an
// ordering only where two agents of a species share a cell: about a sixth of
// the sheep at the workloads' densities, and of those only the ones on grown
// grass or next to a wolf.  So a move sets "a sheep / a second sheep / a wolf /
// a second wolf" in four bits of its cell by LDS atomics, every agent whose
// cell is not contested decides by itself, and the few others (the contested
// list) post their (draw, slot) keys by atomicMin into a small hash table of
// (cell, kind) entries in LDS.  The outcome is the one of posting every key.
// A list that does not fit the table uses the model's claim table in global
// memory for that step, and leaves it all-ones again.
//
// Slots are handled in rows of 64 (one wave instruction, one 64-bit mask per
// property): alive, eaten, breeding, starving, born in this launch.  Sheep rows
// fill the row arrays from the front, wolf rows from the back, so the two
// species share the space.  A step, with a workgroup barrier after each part:
//   A  move      each row: draw, move, set the cell's occupancy bits;
//   B  eat       each row: uncontested outcomes, energy, breeding and starving
//                masks; contested agents are listed;
//   B1 post      the listed agents post their keys;
//   B2 settle    ... and read them back: outcomes, masks;
//   S  scan      a thread per row: prefix sums of the rows' breeders and free slots
//                (the other half of the waves: the step's dead);
//   C  renew     a thread per child: the j-th free slot takes the child of the
//                j-th breeder; a thread per row, of the other half of the waves:
//                the next alive mask.
// What bounds a step is the latency of its six barrier-separated parts (under
// 1 us each for one workgroup, whatever the model's size) and, for large
// models, the instructions per row: 4096 models of 32 x 32 to 256 x 256 cells x
// 50 steps take 7.5 ms, the smaller ones two or four to a CU (50.4 ms by passes
// over global memory); 64 x 64 cells x 200 steps take 1.02 ms (6.36 ms by three
// launches a step).  The busiest wave sets a part's time, so what does not
// need the same rows goes to the other half of the waves (1.02 ms against 1.15
// with all of it on the first ones).
#pragma once

#include "rng.hpp"
#include "scan.hpp"
#include "wave.hpp"

namespace abm {
namespace {

constexpr int kChipThreads = 1024;            // of the largest workgroup
constexpr int32_t kChipSide = 256;            // positions are 8 + 8 bits
constexpr int32_t kChipReadyMax = 254;        // the last step, past the base, that a regrowth byte holds
constexpr int32_t kChipFar = 255;             // ... of a cell grown later: the global array has the step
constexpr int32_t kChipMaxR = 200;            // leaves 54 steps at least between two rebasings
constexpr int32_t kChipMaxGain = 8192;
constexpr int32_t kChipEnergyMax = 16384;     // a 16-bit energy above it ends the on-chip run
constexpr uint32_t kChipNoOwner = 0xFFFFFFFFu;

// What a workgroup of T threads works with.
template <int T>
struct ChipSize {
    static constexpr int32_t kWaves = T / 64;
    static constexpr int32_t kHash = T;              // entries of the contested table
    static constexpr int32_t kHashBits = T == 1024 ? 10 : (T == 512 ? 9 : 8);
    static constexpr int32_t kPosts = T + T / 2;     // a longer list (1 entry or fewer each) may not fit it
    static constexpr int32_t kList = T;              // contested agents listed in LDS (the rest in scratch)
    static constexpr int32_t kMaxRows = T / 2;       // a thread of half the waves per row
    static constexpr int kKeeper = T - 64;           // the thread that keeps the statistics
    static_assert(kHash == 1 << kHashBits, "the hash yields kHashBits bits");
};

// Bytes of LDS besides the rows, and per row of 64 slots.
template <int T>
__host__ __device__ __forceinline__ int64_t chip_fixed_bytes(int64_t cells) {
    const int64_t occ = (cells + 31) / 32 * 16, rdy = (cells + 15) / 16 * 16;
    return occ + rdy + int64_t(ChipSize<T>::kHash) * 12 + int64_t(ChipSize<T>::kList) * 4 + 8;
}
template <class E>
__host__ __device__ __forceinline__ int64_t chip_row_bytes() {
    return 6 * 8 + 4 + 64 * (2 + int64_t(sizeof(E)));
}

// What a launch keeps of a model in the workgroup's static LDS.
struct ChipShared {
    int32_t rows[2][2];          // rows in use per species, by step parity
    uint32_t wsum[kChipThreads / 64];
    int32_t n_list, over, bad, armed;
    int32_t live[2];             // live agents per species
    int32_t eaten, starved[2], grass;
    int32_t mark[2], max_rows[2];
};

// The position of the r-th (0-based) set bit of w, which has more than r.
__device__ __forceinline__ int32_t select_bit64(uint64_t w, int32_t r) {
    uint32_t v = uint32_t(w);
    int32_t base = 0, c = __popc(v);
    if (r >= c) {
        r -= c;
        v = uint32_t(w >> 32);
        base = 32;
    }
#pragma unroll
    for (int h = 16; h >= 1; h >>= 1) {
        const uint32_t low = v & ((1u << h) - 1u);
        c = __popc(low);
        const bool up = r >= c;
        r -= up ? c : 0;
        v = up ? v >> h : low;
        base += up ? h : 0;
    }
    return base;
}

// The lowest k set bits of w (all of them if k is at least their number).
__device__ __forceinline__ uint64_t lowest_bits64(uint64_t w, int32_t k) {
    if (k <= 0) return 0ull;
    if (k >= int32_t(__popcll(w))) return w;
    return w & ((1ull << select_bit64(w, k)) - 1ull);
}

__device__ __forceinline__ uint64_t row_in_cap(int32_t cap, int32_t r) {
    const int32_t left = cap - r * 64;
    return left <= 0 ? 0ull : (left >= 64 ? ~0ull : (1ull << left) - 1ull);
}

// The species' one of two values (a subscript that is not a constant would put
// the pair in memory).
template <class T>
__device__ __forceinline__ T pick(const T (&a)[2], int s) {
    return s ? a[1] : a[0];
}

// A model on the chip, T threads.  V: its view (parameters and global arrays); E: the
// type of an energy in LDS (int16_t, with a bound that ends the run, or
// int32_t).  COUNTDOWN: the grass array holds countdowns instead of the steps
// at which cells are grown.
template <int T, class V, class E, bool COUNTDOWN>
struct Chip : ChipSize<T> {
    using Z = ChipSize<T>;
    const V& v;
    ChipShared& sh;
    int32_t cells, R_rows;       // rows that fit
    uint32_t* occ;
    uint8_t* rdy;
    uint64_t *alive, *eaten, *breed, *starve, *born;   // alive: two buffers by step parity
    uint32_t* pre;               // per row in use: breeders << 16 | free slots before it
    uint16_t* pos;
    E* en;
    uint64_t* hval;
    uint32_t *hown, *list;
    int32_t* spill;              // global: contested agents past the list
    int32_t first;               // step at which the run began
    int tid, lane, wave;

    __device__ __forceinline__ Chip(const V& view, ChipShared& shared, char* lds, int64_t bytes,
                                    int32_t* scratch)
        : v(view), sh(shared), spill(scratch) {
        tid = threadIdx.x;
        lane = tid & 63;
        wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        cells = v.W * v.H;
        R_rows = min(int32_t((bytes - chip_fixed_bytes<T>(cells)) / chip_row_bytes<E>()),
                     Z::kMaxRows);
        char* p = lds;
        hval = reinterpret_cast<uint64_t*>(p);
        p += Z::kHash * 8;
        alive = reinterpret_cast<uint64_t*>(p);
        p += 2 * 8 * int64_t(R_rows);
        eaten = reinterpret_cast<uint64_t*>(p);
        p += 8 * int64_t(R_rows);
        breed = reinterpret_cast<uint64_t*>(p);
        p += 8 * int64_t(R_rows);
        starve = reinterpret_cast<uint64_t*>(p);
        p += 8 * int64_t(R_rows);
        born = reinterpret_cast<uint64_t*>(p);
        p += 8 * int64_t(R_rows);
        // (the 16-byte aligned cell arrays first among the rest)
        p = lds + ((p - lds + 15) & ~int64_t(15));
        occ = reinterpret_cast<uint32_t*>(p);
        p += (int64_t(cells) + 31) / 32 * 16;
        rdy = reinterpret_cast<uint8_t*>(p);
        p += (int64_t(cells) + 15) / 16 * 16;
        hown = reinterpret_cast<uint32_t*>(p);
        p += Z::kHash * 4;
        list = reinterpret_cast<uint32_t*>(p);
        p += Z::kList * 4;
        en = reinterpret_cast<E*>(p);
        p += 64 * int64_t(sizeof(E)) * R_rows;
        pos = reinterpret_cast<uint16_t*>(p);
        p += 64 * 2 * int64_t(R_rows);
        p = lds + ((p - lds + 3) & ~int64_t(3));
        pre = reinterpret_cast<uint32_t*>(p);          // R_rows + 1
    }

    __device__ __forceinline__ int32_t row_at(int s, int32_t r) const { return s ? R_rows - 1 - r : r; }
    __device__ __forceinline__ int32_t cell_of(uint32_t p) const {
        return int32_t(p >> 8) * v.W + int32_t(p & 255u);
    }

    __device__ __forceinline__ void clear_cells() {
        uint4* o = reinterpret_cast<uint4*>(occ);
        for (int32_t i = tid; i < (cells + 31) / 32; i += T) o[i] = uint4{0, 0, 0, 0};
    }
    __device__ __forceinline__ void clear_table() {
        for (int32_t i = tid; i < Z::kHash; i += T) {
            hval[i] = ~0ull;
            hown[i] = kChipNoOwner;
        }
    }

    // Steps from `base` on until a cell is grown, by the global value g (a cell
    // that has not been eaten since the run began).
    __device__ __forceinline__ int32_t far_from(int32_t g, int32_t base) const {
        return max(g, 0) - (COUNTDOWN ? base - first : base);
    }
    // ... as a regrowth byte.
    __device__ __forceinline__ uint32_t ready_byte(int32_t rel) const {
        return uint32_t(min(max(rel, 0), kChipFar));
    }

    // Reads the model's state at step t0.  False if it does not fit the chip
    // form (then nothing has changed).
    __device__ __forceinline__ bool load(int32_t t0) {
        first = t0;
        if (tid == 0) {
            sh.bad = 0;
            sh.armed = 0;
            sh.n_list = 0;
            sh.over = 0;
            sh.mark[0] = sh.mark[1] = 0;
            sh.live[0] = sh.live[1] = 0;
            sh.eaten = sh.grass = 0;
            sh.starved[0] = sh.starved[1] = 0;
        }
        __syncthreads();
        bool bad = false;
        for (int32_t i = tid; i < (cells + 3) / 4; i += T) {
            uint32_t w = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int32_t c = 4 * i + q;
                w |= (c < cells ? ready_byte(far_from(v.ready[c], t0)) : 0u) << (8 * q);
            }
            reinterpret_cast<uint32_t*>(rdy)[i] = w;
        }
        // marks: 1 + the last row with a live agent
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int32_t n = (pick(v.cap, s) + 63) / 64;
            int32_t top = 0;
            constexpr int kAhead = 8;
            for (int32_t r0 = wave; r0 < n; r0 += Z::kWaves * kAhead) {
                int32_t a[kAhead];
#pragma unroll
                for (int q = 0; q < kAhead; ++q) {
                    const int32_t r = r0 + q * Z::kWaves, i = r * 64 + lane;
                    a[q] = r < n && i < pick(v.cap, s) ? pick(v.al, s)[i] : 0;
                }
#pragma unroll
                for (int q = 0; q < kAhead; ++q)
                    if (__ballot(a[q] != 0)) top = r0 + q * Z::kWaves + 1;
            }
            if (lane == 0) atomicMax(&sh.mark[s], top);
        }
        __syncthreads();
        const int32_t rs = sh.mark[0], rw = sh.mark[1];
        if (rs + rw > R_rows) return false;            // (uniform: read from LDS)
        for (int32_t i = tid; i < R_rows; i += T) {
            alive[i] = 0;
            alive[R_rows + i] = 0;
            born[i] = 0;
        }
        clear_cells();
        clear_table();
        __syncthreads();
        for (int32_t q = wave; q < rs + rw; q += Z::kWaves) {
            const int s = q >= rs;
            const int32_t r = s ? q - rs : q, i = r * 64 + lane, at = row_at(s, r);
            const bool in = i < pick(v.cap, s);
            const int32_t x = in ? pick(v.x, s)[i] : 0, y = in ? pick(v.y, s)[i] : 0, e = in ? pick(v.e, s)[i] : 0;
            const bool on = in && pick(v.al, s)[i] != 0;
            // live agents on the grid, their energies in range (what a dead slot
            // holds is not read before a child is put there)
            bad |= on && (uint32_t(x) >= uint32_t(v.W) || uint32_t(y) >= uint32_t(v.H));
            if (sizeof(E) == 2) bad |= on && (e > kChipEnergyMax || e < -kChipEnergyMax);
            pos[at * 64 + lane] = uint16_t(uint32_t(y) << 8 | (uint32_t(x) & 255u));
            en[at * 64 + lane] = E(e);
            const uint64_t m = __ballot(on);
            if (lane == 0) {
                alive[at] = m;
                atomicAdd(&sh.live[s], int32_t(__popcll(m)));
            }
        }
        if (__ballot(bad) && lane == 0) sh.bad = 1;
        if (tid < 2) {
            sh.rows[0][tid] = tid ? rw : rs;
            sh.max_rows[tid] = tid ? rw : rs;
        }
        __syncthreads();
        return sh.bad == 0;
    }

    // Regrowth bytes from base `from` to base `to`; cells eaten since `from`
    // hold R or more and go to the global array (COUNTDOWN: the array is only
    // written at the end).
    __device__ __forceinline__ void rebase(int32_t from, int32_t to) {
        for (int32_t i = tid; i < (cells + 3) / 4; i += T) {
            uint32_t w = reinterpret_cast<uint32_t*>(rdy)[i], out = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int32_t rel = int32_t((w >> (8 * q)) & 255u), c = 4 * i + q;
                if (rel == kChipFar) {
                    out |= ready_byte(far_from(v.ready[c], to)) << (8 * q);
                    continue;
                }
                if (!COUNTDOWN && rel >= v.R && c < cells) v.ready[c] = from + rel;
                out |= ready_byte(rel - (to - from)) << (8 * q);
            }
            reinterpret_cast<uint32_t*>(rdy)[i] = out;
        }
    }

    // Writes the state back after the last step (rows[] of its parity), at
    // step t with base `base`.
    __device__ __forceinline__ void store(int32_t base, int32_t t, int par, const int32_t (&rows0)[2]) {
        for (int32_t i = tid; i < (cells + 3) / 4; i += T) {
            const uint32_t w = reinterpret_cast<uint32_t*>(rdy)[i];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int32_t rel = int32_t((w >> (8 * q)) & 255u), c = 4 * i + q;
                if (c >= cells) continue;
                if (COUNTDOWN) {
                    const int32_t left = rel == kChipFar ? far_from(v.ready[c], t) : rel - (t - base);
                    v.ready[c] = left > 0 ? left : 0;
                } else if (rel >= v.R && rel != kChipFar) {
                    v.ready[c] = base + rel;
                }
            }
        }
        const int32_t ms = sh.max_rows[0], mw = sh.max_rows[1];
        for (int32_t q = wave; q < ms + mw; q += Z::kWaves) {
            const int s = q >= ms;
            const int32_t r = s ? q - ms : q, i = r * 64 + lane, at = row_at(s, r);
            const bool open = r < sh.rows[par][s];     // (rows past it hold no live agent)
            const bool on = open && ((alive[par * R_rows + at] >> lane) & 1);
            const bool child = (born[at] >> lane) & 1;
            // (a slot that held no agent in this run keeps its fields)
            int32_t* const al = pick(v.al, s) + i;
            const int32_t was = i < pick(v.cap, s) && r < pick(rows0, s) ? *al : 0;
            if (i >= pick(v.cap, s) || (was == 0 && !child)) continue;
            const uint32_t p = pos[at * 64 + lane];
            pick(v.x, s)[i] = int32_t(p & 255u);
            pick(v.y, s)[i] = int32_t(p >> 8);
            pick(v.e, s)[i] = int32_t(en[at * 64 + lane]);
            if (!on)
                *al = 0;
            else if (child || was == 2)                // (2 marks an eaten sheep in the other paths)
                *al = 1;
        }
    }

    // ---- contested cells: kind 0 grass, 1 prey, 2 eater
    __device__ __forceinline__ uint64_t key(uint64_t skey, int32_t slot, uint32_t purpose) const {
        return (uint64_t(draw(skey, uint32_t(slot), purpose)) << 32) | uint32_t(slot);
    }
    __device__ __forceinline__ uint32_t hash(uint32_t id) const {
        return (id * 2654435761u) >> (32 - Z::kHashBits);
    }
    __device__ __forceinline__ void post(uint32_t id, uint64_t k) {
        uint32_t h = hash(id);
        for (int probe = 0; probe < 64; ++probe) {
            const uint32_t o = atomicCAS(&hown[h], kChipNoOwner, id);
            if (o == kChipNoOwner || o == id) {
                claim_min_lds(&hval[h], k);
                return;
            }
            h = (h + 1) & (Z::kHash - 1);
        }
        sh.over = 1;
    }
    __device__ __forceinline__ uint64_t posted(uint32_t id) const {
        uint32_t h = hash(id);
        for (int probe = 0; probe < 64; ++probe) {
            if (hown[h] == id) return hval[h];
            h = (h + 1) & (Z::kHash - 1);
        }
        return ~0ull;
    }
    __device__ __forceinline__ uint32_t listed(int32_t q) const {
        uint32_t w = list[q < Z::kList ? q : 0];
        if (q >= Z::kList) w = uint32_t(spill[q - Z::kList]);
        return w;
    }

    // One step t of parity `par` (regrowth base `base`).  True if the run can
    // go on the chip (uniform).  `count`: keep the statistics' counts.
    __device__ __forceinline__ bool step(uint32_t t, int32_t base, int par, bool count) {
        const uint64_t skey = stream_key(v.seed, t);
        const uint32_t T0 = __builtin_amdgcn_readfirstlane(v.T[0]), T1 = __builtin_amdgcn_readfirstlane(v.T[1]);
        const int32_t rs = __builtin_amdgcn_readfirstlane(sh.rows[par][0]);
        const int32_t rw = __builtin_amdgcn_readfirstlane(sh.rows[par][1]);
        const int32_t rows = rs + rw;
        uint64_t* const now = alive + par * R_rows;
        uint64_t* const next = alive + (par ^ 1) * R_rows;
        // ---- A: move
        for (int32_t q = wave; q < rows; q += Z::kWaves) {
            const int s = q >= rs;
            const int32_t r = s ? q - rs : q, at = row_at(s, r);
            if (!((now[at] >> lane) & 1)) continue;
            const uint32_t p = pos[at * 64 + lane];
            const uint32_t d = draw(skey, uint32_t(r * 64 + lane), s ? kWolfMove : kSheepMove) >> 29;
            const int32_t x = wrap_step(int32_t(p & 255u), int32_t((kDxPacked >> (2 * d)) & 3u) - 1, v.W);
            const int32_t y = wrap_step(int32_t(p >> 8), int32_t((kDyPacked >> (2 * d)) & 3u) - 1, v.H);
            pos[at * 64 + lane] = uint16_t(uint32_t(y) << 8 | uint32_t(x));
            const int32_t c = y * v.W + x;
            const uint32_t one = (s ? 4u : 1u) << (4 * (c & 7));
            const uint32_t had = atomicOr(&occ[c >> 3], one);
            if (had & one) atomicOr(&occ[c >> 3], one << 1);
        }
        __syncthreads();
        // ---- B: eat where the cell is not contested, list the others
        const int32_t now_rel = int32_t(t) - base;
        uint32_t ate = 0;
        bool hot = false;                              // an energy near the end of its type
        for (int32_t q = wave; q < rows; q += Z::kWaves) {
            const int s = q >= rs;
            const int32_t r = s ? q - rs : q, at = row_at(s, r), i = r * 64 + lane;
            const bool on = (now[at] >> lane) & 1;
            const int32_t c = on ? cell_of(pos[at * 64 + lane]) : 0;
            const uint32_t nib = occ[c >> 3] >> (4 * (c & 7));
            int32_t e = int32_t(en[at * 64 + lane]) - 1;
            bool gone = false, contested = false, grown = false;
            if (s == 0) {
                grown = int32_t(rdy[c]) <= now_rel;
                const bool multi = nib & 2u, wolf = nib & 4u;
                contested = on && multi && (grown || wolf);
                const bool eats = on && grown && !multi;
                gone = on && wolf && !multi;
                if (eats) rdy[c] = uint8_t(now_rel + v.R);
                e += eats ? v.gain[0] : 0;
                ate += eats ? 1u : 0u;
            } else {
                contested = on && (nib & 8u) && (nib & 1u);
                e += (nib & 8u) || !(nib & 1u) ? 0 : v.gain[1];
            }
            if (on) en[at * 64 + lane] = E(e);
            hot |= on && e > kChipEnergyMax;
            const bool settled = on && !contested && !gone;
            const bool breeds = settled && e > 0 &&
                                draw(skey, uint32_t(i), s ? kWolfBreed : kSheepBreed) < pick(v.T, s);
            const uint64_t mg = __ballot(gone), mb = __ballot(breeds), md = __ballot(settled && e < 0);
            const uint64_t mc = __ballot(contested);
            if (lane == 0) {
                eaten[at] = mg;
                breed[at] = mb;
                starve[at] = md;
            }
            if (mc) {
                int32_t n0 = 0;
                if (lane == 0) n0 = atomicAdd(&sh.n_list, int32_t(__popcll(mc)));
                n0 = __builtin_amdgcn_readfirstlane(n0) + int32_t(lane_rank(mc));
                if (contested) {
                    const uint32_t w = uint32_t(at * 64 + lane) | (s ? 1u << 20 : 0u) |
                                       (grown ? 1u << 21 : 0u) | (nib & 4u ? 1u << 22 : 0u);
                    if (n0 < Z::kList) list[n0] = w; else spill[n0 - Z::kList] = int32_t(w);
                }
            }
        }
        __syncthreads();
        const int32_t n_list = __builtin_amdgcn_readfirstlane(sh.n_list);
        bool global = false;
        if (n_list > 0) {
            // ---- B1: post
            for (int32_t q = tid; q < n_list && n_list <= Z::kPosts; q += T) {
                const uint32_t w = listed(q);
                const int32_t at = int32_t(w & 0xFFFFFu);
                const bool wolf = w & (1u << 20);
                const int32_t i = wolf ? (R_rows - 1 - (at >> 6)) * 64 + (at & 63) : at;
                const uint32_t c = uint32_t(cell_of(pos[at]));
                if (wolf) {
                    post(3 * c + 2, key(skey, i, kWolfEatKey));
                } else {
                    if (w & (1u << 21)) post(3 * c, key(skey, i, kSheepGrassKey));
                    if (w & (1u << 22)) post(3 * c + 1, key(skey, i, kSheepPreyKey));
                }
            }
            __syncthreads();
            global = n_list > Z::kPosts || __builtin_amdgcn_readfirstlane(sh.over) != 0;
            if (global) post_global(skey, n_list);
            // ---- B2: settle
            for (int32_t q = tid; q < n_list; q += T) {
                const uint32_t w = listed(q);
                const int32_t at = int32_t(w & 0xFFFFFu);
                const bool wolf = w & (1u << 20);
                const int32_t i = wolf ? (R_rows - 1 - (at >> 6)) * 64 + (at & 63) : at;
                const int32_t c = cell_of(pos[at]);
                int32_t e = int32_t(en[at]);
                bool gone = false;
                auto best = [&](int kind) {
                    return global ? ld_claim(v.claims + 3 * int64_t(c) + kind) : posted(uint32_t(3 * c + kind));
                };
                if (wolf) {
                    if (best(2) == key(skey, i, kWolfEatKey)) e += v.gain[1];
                } else {
                    if ((w & (1u << 21)) && best(0) == key(skey, i, kSheepGrassKey)) {
                        e += v.gain[0];
                        rdy[c] = uint8_t(now_rel + v.R);
                        ++ate;
                    }
                    gone = (w & (1u << 22)) && best(1) == key(skey, i, kSheepPreyKey);
                }
                en[at] = E(e);
                hot |= e > kChipEnergyMax;
                const uint32_t bit = 1u << (at & 31);
                // (the three masks lie behind each other)
                uint32_t* const me = reinterpret_cast<uint32_t*>(eaten) +
                                     (gone ? 0 : (e > 0 ? 2 : 4) * R_rows);
                const bool set = gone || e < 0 ||
                                 (e > 0 && draw(skey, uint32_t(i), wolf ? kWolfBreed : kSheepBreed) <
                                               (wolf ? T1 : T0));
                if (set) atomicOr(&me[at >> 5], bit);
            }
            __syncthreads();
        }
        if (global)                                    // (every read is behind the barrier)
            for (int32_t q = tid; q < n_list; q += T) {
                uint64_t* cw = v.claims + 3 * int64_t(cell_of(pos[listed(q) & 0xFFFFFu]));
                rearm(cw);
                rearm(cw + 1);
                rearm(cw + 2);
            }
        if (count) {
            const int32_t n = wave_incl_sum(int32_t(ate));
            if (lane == 63 && n) atomicAdd(&sh.grass, n);
        }
        if (sizeof(E) == 2 && __ballot(hot) && lane == 0) sh.bad = 1;
        // ---- S: the rows' breeders and free slots, and the step's dead
        // (the second half of the waves counts the dead meanwhile)
        uint64_t br = 0, f = 0;
        if (tid < rows) {
            const int rs_s = tid >= rs;
            const int32_t r = rs_s ? tid - rs : tid, row = row_at(rs_s, r);
            br = breed[row];
            f = (~now[row] | eaten[row]) & row_in_cap(pick(v.cap, rs_s), r);
        }
        const uint32_t mine = uint32_t(__popcll(br)) << 16 | uint32_t(__popcll(f));
        const uint32_t incl = uint32_t(wave_incl_sum(int32_t(mine)));
        if (wave >= Z::kWaves / 2 && (wave - Z::kWaves / 2) * 64 < rows) {
            const int32_t q = tid - T / 2;
            const int s = q >= rs;
            const int32_t row = row_at(s, s ? q - rs : q);
            const uint64_t gone = q < rows ? eaten[row] : 0ull, dead = q < rows ? starve[row] : 0ull;
            if (__ballot((gone | dead) != 0)) {
                const int32_t g = wave_incl_sum(int32_t(__popcll(gone)));
                const int32_t d0 = wave_incl_sum(s ? 0 : int32_t(__popcll(dead)));
                const int32_t d1 = wave_incl_sum(s ? int32_t(__popcll(dead)) : 0);
                if (lane == 63) {
                    if (g) atomicAdd(&sh.eaten, g);
                    if (d0) atomicAdd(&sh.starved[0], d0);
                    if (d1) atomicAdd(&sh.starved[1], d1);
                }
            }
        }
        if (lane == 63) sh.wsum[wave] = incl;
        if (tid < 2) sh.rows[par ^ 1][tid] = 0;
        __syncthreads();
        {
            const uint32_t w = lane < Z::kWaves ? sh.wsum[lane] : 0u;
            const int32_t wi = wave_incl_sum(int32_t(w));
            const uint32_t before = wave ? uint32_t(__builtin_amdgcn_readlane(wi, wave - 1)) : 0u;
            if (tid < rows) pre[tid] = before + incl - mine;
            if (tid == rows - 1) pre[rows] = before + incl;
            if (rows == 0 && tid == 0) pre[0] = 0;
        }
        __syncthreads();
        // ---- C: renew
        const uint32_t ps = __builtin_amdgcn_readfirstlane(pre[rs]);
        const uint32_t pt = __builtin_amdgcn_readfirstlane(pre[rows]);
        const int32_t nb[2] = {int32_t(ps >> 16), int32_t((pt - ps) >> 16)};
        const int32_t nf[2] = {int32_t(ps & 0xFFFFu), int32_t((pt - ps) & 0xFFFFu)};
        int32_t births[2], end[2];
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int32_t n = s ? rw : rs;
            const int32_t past = pick(v.cap, s) > n * 64 ? pick(v.cap, s) - n * 64 : 0;   // free slots past the rows
            births[s] = nb[s] < nf[s] + past ? nb[s] : nf[s] + past;
            const int32_t more = births[s] > nf[s] ? births[s] - nf[s] : 0;
            end[s] = n + (more + 63) / 64;
        }
        // rows once used keep their place (their dead slots' fields are written
        // back at the end); births past what is left go to global memory
        const int32_t had[2] = {__builtin_amdgcn_readfirstlane(sh.max_rows[0]),
                                __builtin_amdgcn_readfirstlane(sh.max_rows[1])};
        const bool fits = max(end[0], had[0]) + max(end[1], had[1]) <= R_rows;
        if (!fits) {
            end[0] = min(end[0], had[0]);
            end[1] = min(end[1], had[1]);
        }
        for (int32_t j = tid; j < births[0] + births[1]; j += T) {
            const int s = j >= births[0];
            const int32_t jj = s ? j - births[0] : j;
            const int32_t first = s ? rs : 0, n = s ? rw : rs;
            const uint32_t p0 = s ? ps : 0u;
            // the rows of breeder jj and of free slot jj: the last with at most jj before it
            int32_t pr = 0, cr = 0;
            for (int32_t h = 512; h >= 1; h >>= 1) {
                if (h >= n) continue;                  // (uniform unless the species differ)
                const int32_t i0 = pr + h, i1 = cr + h;
                const uint32_t w0 = i0 < n ? pre[first + i0] - p0 : 0u;
                const uint32_t w1 = i1 < n ? pre[first + i1] - p0 : 0u;
                pr = i0 < n && int32_t(w0 >> 16) <= jj ? i0 : pr;
                cr = i1 < n && int32_t(w1 & 0xFFFFu) <= jj ? i1 : cr;
            }
            const int32_t pat = row_at(s, pr);
            const int32_t pb = select_bit64(breed[pat], jj - int32_t((pre[first + pr] - p0) >> 16));
            const int32_t parent = pat * 64 + pb;
            const int32_t ep = int32_t(en[parent]), ec = ep >> 1;
            const uint32_t pp = pos[parent];
            en[parent] = E(ep - ec);
            if (jj < pick(nf, s)) {
                const int32_t cat = row_at(s, cr);
                const uint64_t fm = (~now[cat] | eaten[cat]) & row_in_cap(pick(v.cap, s), cr);
                const int32_t slot = cat * 64 + select_bit64(fm, jj - int32_t((pre[first + cr] - p0) & 0xFFFFu));
                pos[slot] = uint16_t(pp);
                en[slot] = E(ec);
            } else {
                const int32_t i = n * 64 + (jj - pick(nf, s));
                if ((i >> 6) < pick(end, s)) {
                    const int32_t slot = row_at(s, i >> 6) * 64 + (i & 63);
                    pos[slot] = uint16_t(pp);
                    en[slot] = E(ec);
                } else {
                    pick(v.x, s)[i] = int32_t(pp & 255u);
                    pick(v.y, s)[i] = int32_t(pp >> 8);
                    pick(v.e, s)[i] = ec;
                    pick(v.al, s)[i] = 1;
                }
            }
        }
        // the next alive masks, and the rows they use, by the second half of the
        // waves (few steps have so many births that those bear children too)
        if (wave >= Z::kWaves / 2 && tid - T / 2 < end[0] + end[1]) {
            const int32_t q = tid - T / 2;
            const int s = q >= end[0];
            const int32_t r = s ? q - end[0] : q, at = row_at(s, r);
            const int32_t first = s ? rs : 0, n = s ? rw : rs;
            const uint32_t p0 = s ? ps : 0u;
            const uint64_t cap = row_in_cap(pick(v.cap, s), r);
            uint64_t add, m = 0;
            if (r < n) {
                const uint64_t al = now[at], g = eaten[at];
                add = lowest_bits64((~al | g) & cap, pick(births, s) - int32_t((pre[first + r] - p0) & 0xFFFFu));
                m = al & ~g & ~starve[at];
            } else {
                add = lowest_bits64(cap, pick(births, s) - pick(nf, s) - (r - n) * 64);
            }
            m |= add;
            next[at] = m;
            if (add) born[at] |= add;
            if (m) atomicMax(&sh.rows[par ^ 1][s], r + 1);
        }
        clear_cells();
        if (n_list > 0) clear_table();
        if (tid == 0) {
            sh.n_list = 0;
            sh.over = 0;
        }
        last_births[0] = births[0];
        last_births[1] = births[1];
        __syncthreads();
        if (tid == 0) {                                // (read again behind the next step's barriers)
            sh.max_rows[0] = max(had[0], end[0]);
            sh.max_rows[1] = max(had[1], end[1]);
        }
        return fits && sh.bad == 0;
    }

    int32_t last_births[2];

    // The contested list's keys into the global claim table (all-ones before;
    // COUNTDOWN: the call's first use makes it so).  A wave's stores and atomics
    // are performed before the barrier that ends each part.
    __device__ __forceinline__ void post_global(uint64_t skey, int32_t n_list) {
        if (COUNTDOWN && sh.armed == 0) {
            for (int64_t w = tid; w < 3 * int64_t(cells); w += T) rearm(v.claims + w);
        }
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        if (tid == 0) sh.armed = 1;
        for (int32_t q = tid; q < n_list; q += T) {
            const uint32_t w = listed(q);
            const int32_t at = int32_t(w & 0xFFFFFu);
            const bool wolf = w & (1u << 20);
            const int32_t i = wolf ? (R_rows - 1 - (at >> 6)) * 64 + (at & 63) : at;
            uint64_t* cw = v.claims + 3 * int64_t(cell_of(pos[at]));
            if (wolf) {
                claim_min(cw + 2, key(skey, i, kWolfEatKey));
            } else {
                if (w & (1u << 21)) claim_min(cw, key(skey, i, kSheepGrassKey));
                if (w & (1u << 22)) claim_min(cw + 1, key(skey, i, kSheepPreyKey));
            }
        }
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
    }
};

// What the caller of run_on_chip keeps per step: live agents at its start and
// its events (thread ChipSize<T>::kKeeper, whose wave has the fewest rows).
struct ChipStats {
    int64_t* row;        // next statistics row, or null
    uint64_t updates;    // live agents summed over the steps' starts
};

// Advances model v from step t0 towards t1 on the chip; returns the step
// reached (t0 if the model does not fit; less than t1 if its rows or energies
// outgrew the chip).  The global state is current when it returns.
template <int T, class E, bool COUNTDOWN, class V>
__device__ __forceinline__ int32_t run_on_chip(const V& v, ChipShared& sh, char* lds, int64_t bytes,
                                               int32_t* scratch, int32_t t0, int32_t t1,
                                               ChipStats* st) {
    Chip<T, V, E, COUNTDOWN> c(v, sh, lds, bytes, scratch);
    if (c.R_rows < 2 || !c.load(t0)) {
        __syncthreads();
        return t0;
    }
    const int32_t rows0[2] = {sh.rows[0][0], sh.rows[0][1]};
    int32_t live[2] = {sh.live[0], sh.live[1]};
    int32_t eaten = 0, grass = 0, starved[2] = {0, 0};
    const bool count = st->row != nullptr;
    int32_t base = t0, t = t0;
    int par = 0;
    bool go = true;
    for (; t < t1 && go; ++t, par ^= 1) {
        if (t - base + v.R > kChipReadyMax) {
            c.rebase(base, t);
            base = t;
            __syncthreads();
        }
        go = c.step(uint32_t(t), base, par, count);
        if (c.tid == ChipSize<T>::kKeeper) {
            const int32_t ne = sh.eaten - eaten, n0 = sh.starved[0] - starved[0],
                          n1 = sh.starved[1] - starved[1];
            st->updates += uint64_t(live[0] + live[1]);
            if (count) {
                int64_t* r = st->row;
                r[0] = live[0];
                r[1] = live[1];
                r[2] = sh.grass - grass;
                r[3] = ne;
                r[4] = c.last_births[0];
                r[5] = c.last_births[1];
                r[6] = n0;
                r[7] = n1;
                st->row += 8;
            }
            live[0] += c.last_births[0] - ne - n0;
            live[1] += c.last_births[1] - n1;
            eaten += ne;
            starved[0] += n0;
            starved[1] += n1;
            grass = sh.grass;
        }
    }
    __syncthreads();                                   // max_rows is current
    c.store(base, t, par, rows0);
    __syncthreads();
    return t;
}

}  // namespace
}  // namespace abm
