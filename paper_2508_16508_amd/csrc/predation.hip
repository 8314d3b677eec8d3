// predation.hip -- abm_predation_init / abm_predation_step: the wolf-sheep-
// grass model of Sec. 5.1 (Fig. 2) on one GPU, one model per launch sequence.
//
// A model whose slots and cells all fit one workgroup's LDS is advanced there,
// a call being one launch (launch_small_predation); what follows is the
// general path.
//
// Inside a call the state is kept in two working forms (converted at the call's
// start and back at its end): grass holds the step at which a cell is grown
// again (grown at step t iff ready <= t), so no per-step regrow pass is needed,
// and a bitmask in the workspace marks the live slots, so the per-step kernels
// read 1 bit per slot instead of the 4-byte alive word and visit only live
// agents.  Each kernel works on tiles of 2048 slots, four slots a thread, whose
// loads and random accesses are in flight together; a slot that is not live
// repeats the block's first load, so nothing branches around a load.
// Step t is three launches (each arrow a grid-wide dependency):
//   K1 move+claim   every live agent moves, pays 1 energy and posts its
//                   packed (step tag, draw, slot) key with a 64-bit atomicMin
//                   into the claim tables of its cell: grass (sheep on grown
//                   cells), prey (sheep) and eater (wolves).
//   K2 eat+breeders each live agent compares its keys with the reduced table
//                   entries (grass winner, eaten sheep, eating wolf), applies
//                   the energy gain and marks an eaten sheep alive = 2, then
//                   decides whether it breeds; the tile's breeders and its
//                   slots free for births (empty, or eaten this step) are
//                   ranked by the single-pass scan on two chains at once, the
//                   breeders compacted into an ascending list and the tile's
//                   free-slot prefix kept for K3.
//   K3 breed+die    the free slot of rank j < #breeders PULLS its child from
//                   breeder j (cell, half the energy) while the parent keeps
//                   the rest; live agents with negative energy die; at the end
//                   of a tag period the claim tables are re-armed (each
//                   workgroup streams its slice; within a period the falling
//                   tags make older words lose, see claim_key).
// Blocks past the last one holding a live agent (the mark K3 leaves for the
// next step) skip their work: they hold no agent, K2's scans stop below them,
// and K3 computes their free-slot prefixes from the totals.
// With multi_prey, K1 instead pushes every live sheep and wolf onto a list of
// its cell (64-bit atomicExch on the prey / eater words, which then hold list
// heads), and K1b, between K1 and K2, pairs the r-th wolf of each cell (eat
// key order) with the r-th sheep (prey key order): the wolf gains, the sheep
// is marked alive = 2 (eaten, still to take part in the grass rule of K2).
// Pulling into the free slot (rather than the parent pushing into some later
// tile) keeps every slot written by one thread.
#include <hip/hip_runtime.h>

#include "abm.h"
#include "common.hpp"
#include "rng.hpp"
#include "scan.hpp"

namespace abm {
namespace {

constexpr int kBlock = 256;                       // threads of the element-wise kernels
constexpr int kOwners = 64;                       // threads that own a tile's bitmask words
constexpr int64_t kTile = int64_t(kOwners) * 32;  // 2048 slots: one bitmask word per owner
constexpr uint32_t kTagBits = 4;                  // claim-key tag: periods of 14 steps
// Threads of a workgroup, four slots of a tile each.  Live agents crowd the low
// tiles (children take the lowest free slots), so the tiles must be small for
// the work to reach every CU, and their threads many: the chain of dependent
// random accesses of an agent bounds the step.  In us per step, with tiles of
// 8192 slots, whose live slots 1024 threads took from a list, and now: 300^2
// cells 70 and 33, 700^2 87 and 36, 2048^2 with 10 % sheep 106 and 63, with
// 38 % (2 M agents at first, where the 26 G atomics a second bound K1 and the
// lines of the claim table K2) 126 and 120.
constexpr int kThreads = 512;
constexpr int kThreadWaves = kThreads / 64;
constexpr int kPerThread = int(kTile) / kThreads;
// The workgroups of a species take one tile each up to kSingleTiles (2 M
// slots), and kTilesPerBlock tiles beyond: those are empty in most states, and
// workgroups that only find that out cost their dispatch (16 M slots: 8192).
constexpr uint32_t kSingleTiles = 1024, kTilesPerBlock = 8;
constexpr int kBlockWords = kOwners * int(kTilesPerBlock);   // bitmask words, one a thread
static_assert(kBlockWords == kThreads, "a thread per bitmask word of a block");
// header words of the free-slot totals (words 4 and 5 are unused by the
// common layout)
constexpr int kHdrFreeA = 4, kHdrFreeB = 5;
// words 6-21: the block marks of even and odd steps, two species each, each
// spread over four words (a workgroup raises the one of its number: atomics on
// one address serialise)
constexpr int kHdrMark = 6, kMarkLanes = 4;
static_assert(kHdrFreeA > kHdrCountB && kHdrMark + 4 * kMarkLanes <= kHdrError,
              "header word clash");
static_assert(kThreadWaves >= 2 * kLevels, "the dual-chain prefix needs 2 kLevels waves");
constexpr uint64_t kNoClaim = ~0ull;

// Offsets of the eight neighbours, indexed by dir = draw >> 29, packed as
// (offset + 1) in two bits per direction:
//   dir: 0 (-1,-1) 1 (0,-1) 2 (1,-1) 3 (-1,0) 4 (1,0) 5 (-1,1) 6 (0,1) 7 (1,1)
constexpr uint32_t kDxPacked = 0x9224u;
constexpr uint32_t kDyPacked = 0xA940u;

enum StatCol : int {
    kLiveS = 0, kLiveW, kGrassEaten, kSheepEaten, kBirthsS, kBirthsW, kStarvedS, kStarvedW
};

struct Species {
    int32_t* x;
    int32_t* y;
    int32_t* e;
    int32_t* alive;
};

struct StepArgs {
    int32_t W, H, R, gain_s, gain_w;
    uint32_t T_s, T_w, seed;
    int64_t cap_s, cap_w;
    int32_t* ready;       // grass: step at which each cell is grown again
    Species sp[2];        // 0 sheep, 1 wolves
    uint32_t* bits[2];    // live-slot bitmasks
    int64_t G;            // cells
    uint64_t* claims;     // three words per cell c, at 3 c: grass (the lowest key
                          // of a sheep on the grown cell), prey (lowest sheep
                          // key), eater (lowest wolf key); together in one line
    uint32_t sb;          // slot bits of a claim key (see claim_key)
    uint64_t tag_hi;      // this step's tag, in place
    uint64_t tag_mask;    // the tag field
    int32_t rearm;        // K3 re-arms the whole table (the tag period ends)
    int64_t* stats;       // this step's row of 8, or null
    int64_t* acc;         // kAccCounters x kAccLanes spread accumulators: per counter, lanes
                          // [0, 128) for even steps of a call and [128, 256) for odd ones
    int32_t acc_par;      // this step's half (0 or 128)
    int64_t* fold_row;    // stats row of the previous step, folded by K1 (or null)
    uint32_t step;
    uint64_t* status;
    uint64_t* err;        // set when a wait of the scans gives up
    unsigned long long* updates;   // live agents are added to it (or null)
    EpochArg epoch;
    int32_t* blist[2];    // breeder lists
    int64_t* d_nb[2];     // breeder counts
    int64_t* d_nf[2];     // free-slot counts (this step's births are min(nf, nb))
    int32_t* free_pre[2]; // per block: exclusive free-slot prefix, written by K2 for K3
    uint32_t tiles[2];
    uint32_t blocks[2];
    uint32_t turn;          // blocks of a species in turn: 2^turn (see Block)
    uint32_t chain_off[2];  // start of each species' breeder scan chain in the status words
    uint32_t fchain_off[2]; // ... and of its free-slot scan chain
    int32_t multi;          // prey by rank within a cell (K1 builds lists, K1b matches)
    int32_t batch;          // a model of a batch
    uint64_t* mark_rd;      // [2][kMarkLanes] per species: no live agent in a block past the largest
    uint64_t* mark_wr;      // the same for the next step, raised by K3 (cleared by K1)
};

__device__ __forceinline__ int32_t wrap_step(int32_t v, int32_t d, int32_t n) {
    v += d;
    return v < 0 ? n - 1 : (v >= n ? 0 : v);
}

// Cell of a position, or -1 when it lies off the lattice (a live agent is
// always on it in a state produced by this library; the test keeps a bad
// caller-supplied state from indexing outside the grid).
__device__ __forceinline__ int64_t cell_of(int32_t x, int32_t y, int32_t W, int32_t H) {
    return (x >= 0 && x < W && y >= 0 && y < H) ? int64_t(y) * W + x : -1;
}

__device__ __forceinline__ uint64_t agent_key(uint64_t skey, int64_t slot, uint32_t purpose) {
    return (uint64_t(draw(skey, uint32_t(slot), purpose)) << 32) | uint32_t(slot);
}

// A claim word holds (tag, draw, slot) from the high bits down: slot in the
// low sb bits, the 32-bit draw above it and the step's tag on top.  Within a
// step, keys order as (draw, slot), the order of the method's claims.  Tags
// fall from step to step, so a word left by an earlier step of the same
// period (a larger tag) loses to every fresh claim and reads as unclaimed,
// and the table need not be re-armed between the steps of a period; all-ones
// (the re-armed word) carries a tag no step uses.
__device__ __forceinline__ uint64_t claim_key(const StepArgs& a, uint64_t skey, int64_t slot,
                                              uint32_t purpose) {
    return a.tag_hi | (uint64_t(draw(skey, uint32_t(slot), purpose)) << a.sb) | uint64_t(slot);
}

__device__ __forceinline__ bool claimed(const StepArgs& a, uint64_t word) {
    return (word & a.tag_mask) == a.tag_hi;
}

// Slot at the head of a multi-prey list word, or -1 (no push this step).
__device__ __forceinline__ int32_t head_slot(const StepArgs& a, uint64_t word) {
    return claimed(a, word) ? int32_t(word & ~a.tag_mask) : -1;
}

// Block-wide sum of one value per thread, added by thread 0 to this block's
// lane of the spread accumulator of counter `col` in the step's half (128
// lanes per counter and step, so no single address takes every block's
// atomic).  `acc` points at the step's half.
constexpr int kHalfLanes = kAccLanes / 2;
__device__ __forceinline__ void block_add(uint32_t v, int64_t* acc, int col, uint32_t* lds) {
    int64_t* dst = acc + int64_t(col) * kAccLanes + (blockIdx.x & (kHalfLanes - 1));
    const uint32_t w = wave_sum(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = w;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t s = 0;
        for (int i = 0; i < int(blockDim.x >> 6); ++i) s += lds[i];
        if (s) atomicAdd(reinterpret_cast<unsigned long long*>(dst), (unsigned long long)s);
    }
}

// Folds one step's half of the spread accumulators (`acc` points at it)
// into its stats row (the births columns are written by K3) and clears it for
// the step after next.  Any number of whole waves.
__device__ __forceinline__ void fold_stats(int64_t* acc, int64_t* stats) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int col = wave; col < kAccCounters; col += int(blockDim.x >> 6)) {
        int64_t v = 0;
        for (int l = lane; l < kHalfLanes; l += 64) {
            v += acc[col * kAccLanes + l];
            acc[col * kAccLanes + l] = 0;
        }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
        if (lane == 0 && col != kBirthsS && col != kBirthsW) stats[col] = v;
    }
}

// ------------------------------------------------------------------ init
struct InitArgs {
    int32_t W, H, R, gain_s, gain_w;
    uint32_t seed;
    int64_t cap_s, cap_w, n_s0, n_w0, G;
    int32_t* grass;
    Species sp[2];
    uint64_t* claims;  // 3 * G
};

__global__ __launch_bounds__(kBlock) void k_init(InitArgs a) {
    const int64_t i = int64_t(blockIdx.x) * kBlock + threadIdx.x;
    const uint64_t key = stream_key(a.seed, kInitStep);
    if (i < a.G) {
        const uint32_t h = draw(key, uint32_t(i), kGrassGrown);
        a.grass[i] = h < 0x80000000u
                         ? 0
                         : 1 + int32_t(scale(draw(key, uint32_t(i), kGrassCountdown), uint32_t(a.R)));
        a.claims[i] = kNoClaim;
        a.claims[a.G + i] = kNoClaim;
        a.claims[2 * a.G + i] = kNoClaim;
    }
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const int64_t cap = s ? a.cap_w : a.cap_s;
        const int64_t n0 = s ? a.n_w0 : a.n_s0;
        const int32_t gain = s ? a.gain_w : a.gain_s;
        const uint32_t px = s ? kWolfX : kSheepX;
        if (i < cap) {
            int32_t x = 0, y = 0, e = 0, al = 0;
            if (i < n0) {
                x = int32_t(scale(draw(key, uint32_t(i), px), uint32_t(a.W)));
                y = int32_t(scale(draw(key, uint32_t(i), px + 1), uint32_t(a.H)));
                e = int32_t(scale(draw(key, uint32_t(i), px + 2), uint32_t(2 * gain)));
                al = 1;
            }
            a.sp[s].x[i] = x;
            a.sp[s].y[i] = y;
            a.sp[s].e[i] = e;
            a.sp[s].alive[i] = al;
        }
    }
}

__global__ __launch_bounds__(kBlock) void k_fill64(int64_t* p, int64_t n, int64_t v) {
    const int64_t i = int64_t(blockIdx.x) * kBlock + threadIdx.x;
    if (i < n) p[i] = v;
}

// ------------------------------------------------------------------ tiles
// Tile t of a species covers slots [2048 t, 2048 t + 2048) and bitmask words
// [64 t, 64 t + 64).  Bits of slots at or beyond the capacity are always zero.
// A block is what one workgroup takes: one tile, or kTilesPerBlock consecutive
// ones.  The blocks of both species are interleaved, 2^turn of each in turn
// until the shorter chain ends, then the rest, so that the low tiles, where
// children fill the lowest free slots and the live agents gather, are all in
// the first round of resident workgroups; within each chain blocks still run
// in increasing order.  Workgroups go to the eight XCDs in turn, so single
// blocks leave all the sheep to four of them.  Small launches are better with
// eight blocks in turn (us per step: 300^2 cells 31.3 against 32.9, 2048^2 with
// a slot a cell 61.9 against 63.4), large ones, at the atomics' rate, with one
// (2048^2 with four slots a cell, 3072 blocks: 120 against 124).
struct Block {
    int s;            // species
    uint32_t q;       // block within the species' scan chain
    uint32_t words;   // bitmask words, 64 per tile
    int64_t word0;    // the first of them
    int64_t base;     // first slot
};

__host__ __device__ __forceinline__ uint32_t blocks_of(uint32_t tiles) {
    return tiles <= kSingleTiles
               ? tiles
               : kSingleTiles + (tiles - kSingleTiles + kTilesPerBlock - 1) / kTilesPerBlock;
}

__device__ __forceinline__ uint32_t first_tile(uint32_t q) {
    return q < kSingleTiles ? q : kSingleTiles + (q - kSingleTiles) * kTilesPerBlock;
}

// The species' one of a pair (a subscript that is not a constant would put the
// arguments in memory where they are a local copy).
template <class T>
__device__ __forceinline__ T pick(const T (&a)[2], int s) {
    return s ? a[1] : a[0];
}

// Block n of the interleaved order.
__device__ __forceinline__ Block block_of(const StepArgs& a, uint32_t n) {
    const uint32_t low = (1u << a.turn) - 1u;
    const uint32_t m = (a.blocks[0] < a.blocks[1] ? a.blocks[0] : a.blocks[1]) & ~low;
    Block b;
    if (n < 2 * m) {
        b.s = int((n >> a.turn) & 1u);
        b.q = ((n >> (a.turn + 1)) << a.turn) + (n & low);
    } else {
        const uint32_t r = n - 2 * m, rest0 = a.blocks[0] - m;
        b.s = r < rest0 ? 0 : 1;
        b.q = m + (b.s ? r - rest0 : r);
    }
    const uint32_t t = first_tile(b.q), left = (b.s ? a.tiles[1] : a.tiles[0]) - t;
    b.words = kOwners * (b.q < kSingleTiles ? 1u : (left < kTilesPerBlock ? left : kTilesPerBlock));
    b.word0 = int64_t(t) * kOwners;
    b.base = int64_t(t) * kTile;
    return b;
}

// Blocks of species s from which on no agent is alive.
__device__ __forceinline__ uint32_t mark_of(const StepArgs& a, int s) {
    uint64_t m = 0;
#pragma unroll
    for (int l = 0; l < kMarkLanes; ++l) {
        const uint64_t v = a.mark_rd[s * kMarkLanes + l];
        m = v > m ? v : m;
    }
    return uint32_t(m);
}

// The arrays from slot `base` on.
__device__ __forceinline__ Species species_at(const Species& s, int64_t base) {
    return Species{s.x + base, s.y + base, s.e + base, s.alive + base};
}

// Slot (within the block) k of this thread in the tile whose words start at w0
// of the block, and whether its bit is set.
__device__ __forceinline__ uint32_t slot_in_block(uint32_t w0, int k) {
    return w0 * 32u + uint32_t(k) * kThreads + threadIdx.x;
}

__device__ __forceinline__ uint32_t live_of(const StepArgs& a, const Block& b, uint32_t w0) {
    uint32_t word[kPerThread], live = 0;
#pragma unroll
    for (int k = 0; k < kPerThread; ++k)
        word[k] = pick(a.bits, b.s)[b.word0 + (slot_in_block(w0, k) >> 5)];
#pragma unroll
    for (int k = 0; k < kPerThread; ++k) live |= ((word[k] >> (threadIdx.x & 31)) & 1u) << k;
    return live;
}

// Bit `slot` of a block's masks in LDS.
__device__ __forceinline__ void set_bit(uint32_t* masks, uint32_t slot) {
    atomicOr(&masks[slot >> 5], 1u << (slot & 31u));
}

// The slots of word w (of the block) below the capacity.
__device__ __forceinline__ uint32_t word_in_cap(const Block& b, uint32_t w, int64_t cap) {
    const int64_t left = w < b.words ? cap - b.base - int64_t(w) * 32 : 0;
    return left <= 0 ? 0u : low_bits(left < 32 ? uint32_t(left) : 32u);
}

// In a one-model call ready is step + countdown and may wrap; in a batch it is a
// step, or anything that the caller set it to.
__device__ __forceinline__ bool grown(const StepArgs& a, int32_t ready) {
    return a.batch ? ready <= int32_t(a.step) : int32_t(uint32_t(ready) - a.step) <= 0;
}

// Tile-local part of a rank: this thread's exclusive rank of its count c
// (0 <= c < 64) in thread order, and the tile total.  lds holds one word per
// wave.  Two block barriers.
__device__ __forceinline__ uint32_t rank_block(uint32_t c, uint32_t* thread_excl, uint32_t* lds) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t excl = 0, wtot = 0;
#pragma unroll
    for (int b = 0; b < 6; ++b) {
        const uint64_t bal = __ballot((c >> b) & 1u);
        excl += lane_rank(bal) << b;
        wtot += static_cast<uint32_t>(__popcll(bal)) << b;
    }
    __syncthreads();
    if (lane == 0) lds[wave] = wtot;
    __syncthreads();
    uint32_t before = 0, total = 0;
#pragma unroll
    for (int w = 0; w < kThreadWaves; ++w) {
        const uint32_t v = lds[w];
        before += w < wave ? v : 0u;
        total += v;
    }
    *thread_excl = before + excl;
    return total;
}

// Exclusive prefixes of two counts of this tile over two chains at once (the
// hierarchical look-back of the single-pass scan, one chain per group of
// kLevels waves: waves 0-3 walk chain A with count a, waves 4-7 chain B with
// count b).  Needs 2 kLevels waves; lds holds 2 kLevels words.  Two barriers.
__device__ __forceinline__ void hier_prefix2(uint64_t* chain_a, uint64_t* chain_b, uint64_t* err,
                                             uint32_t t, uint32_t T, uint32_t epoch, uint32_t a,
                                             uint32_t b, uint32_t* lds, uint32_t* pre_a,
                                             uint32_t* pre_b) {
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const bool second = wave >= kLevels;
    const int lv = second ? wave - kLevels : wave;
    const uint32_t count = second ? b : a;
    uint32_t part = 0;
    if (wave < 2 * kLevels) {
        uint64_t* level = second ? chain_b : chain_a;
        uint32_t n = T;
        for (int l = 0; l < lv; ++l) {
            level += n;
            n = (n + 63) >> 6;
        }
        const uint32_t g = t >> (6 * lv);
        const uint32_t d = g & 63u;
        const uint32_t pspan = 1u << (6 * (lv + 1));
        const bool publish = (((t & (pspan - 1)) == pspan - 1) || t == T - 1) && lv + 1 < kLevels;
        if (lv == 0 && lane == 0) st_agent(&level[g], pack_status(epoch, kFlagAgg, count));
        uint32_t v = 0;
        if (lane < d || (lane == d && lv > 0 && publish)) {
            const uint32_t idx = g - d + lane;
            v = static_cast<uint32_t>(poll_status(&level[idx], ld_agent(&level[idx]), epoch, err));
        }
        const uint32_t own = (lv == 0) ? count : 0u;
        part = wave_sum(lane < d ? v : 0u);
        if (publish) {
            const uint32_t incl = wave_sum(v) + own;
            if (lane == 0) st_agent(&(level + n)[g >> 6], pack_status(epoch, kFlagAgg, incl));
        }
    }
    __syncthreads();
    if (lane == 0 && wave < 2 * kLevels) lds[wave] = part;
    __syncthreads();
    uint32_t ta = 0, tb = 0;
#pragma unroll
    for (int l = 0; l < kLevels; ++l) {
        ta += lds[l];
        tb += lds[kLevels + l];
    }
    *pre_a = ta;
    *pre_b = tb;
}

// ------------------------------------------------------------------ K1
__device__ __forceinline__ void move_claim(const StepArgs& a, const Block& b, uint32_t* lds) {
    const int s = b.s;
    if (b.q >= mark_of(a, s)) return;   // past the last live agent
    const Species sp = species_at(pick(a.sp, s), b.base);
    const uint32_t base = uint32_t(b.base);
    const uint64_t skey = stream_key(a.seed, a.step);
    uint32_t count = 0;
    for (uint32_t w0 = 0; w0 < b.words; w0 += kOwners) {
        const uint32_t live = live_of(a, b, w0);
        if (__ballot(live != 0u) == 0) continue;   // (the wave's)
        count += __popc(live);
        uint32_t i[kPerThread];
        int32_t c[kPerThread];
        int32_t x[kPerThread], y[kPerThread], e[kPerThread];
#pragma unroll
        for (int k = 0; k < kPerThread; ++k) {
            // (a dead slot's loads go to the block's first: no branch around them)
            i[k] = (live >> k) & 1u ? slot_in_block(w0, k) : 0u;
            x[k] = sp.x[i[k]];
            y[k] = sp.y[i[k]];
            e[k] = sp.e[i[k]];
        }
#pragma unroll
        for (int k = 0; k < kPerThread; ++k) {
            c[k] = -1;
            if (!((live >> k) & 1u)) continue;
            const uint32_t d = draw(skey, base + i[k], s ? kWolfMove : kSheepMove) >> 29;
            x[k] = wrap_step(x[k], int32_t((kDxPacked >> (2 * d)) & 3u) - 1, a.W);
            y[k] = wrap_step(y[k], int32_t((kDyPacked >> (2 * d)) & 3u) - 1, a.H);
            sp.x[i[k]] = x[k];
            sp.y[i[k]] = y[k];
            sp.e[i[k]] = e[k] - 1;
            c[k] = int32_t(cell_of(x[k], y[k], a.W, a.H));
        }
        bool grows[kPerThread];
#pragma unroll
        for (int k = 0; k < kPerThread; ++k)
            grows[k] = s == 0 && c[k] >= 0 && grown(a, a.ready[c[k]]);
#pragma unroll
        for (int k = 0; k < kPerThread; ++k) {
            if (c[k] < 0) continue;
            uint64_t* const cell = a.claims + 3 * int64_t(c[k]);
            if (grows[k])
                atomicMin(reinterpret_cast<unsigned long long*>(cell),
                          (unsigned long long)claim_key(a, skey, base + i[k], kSheepGrassKey));
            if (a.multi) {
                // push slot i onto the list of its cell; the list ends at a word
                // of an earlier step (or all-ones)
                const uint64_t prev =
                    atomicExch(reinterpret_cast<unsigned long long*>(cell + (s ? 2 : 1)),
                               (unsigned long long)(a.tag_hi | uint64_t(base + i[k])));
                pick(a.blist, s)[base + i[k]] = head_slot(a, prev);
            } else {
                atomicMin(reinterpret_cast<unsigned long long*>(cell + (s ? 2 : 1)),
                          (unsigned long long)claim_key(a, skey, base + i[k],
                                                        s ? kWolfEatKey : kSheepPreyKey));
            }
        }
    }
    if (a.stats) block_add(count, a.acc + a.acc_par, s ? kLiveW : kLiveS, lds);
    if (a.updates) {
        const uint32_t v = wave_sum(count);
        if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = v;
        __syncthreads();
        if (threadIdx.x == 0) {
            uint32_t all = 0;
            for (int w = 0; w < kThreadWaves; ++w) all += lds[w];
            if (all) atomicAdd(a.updates, (unsigned long long)all);
        }
    }
}

__global__ __launch_bounds__(kThreads) void k_move_claim(StepArgs a) {
    __shared__ uint32_t lds[kThreadWaves];
    // the previous step's statistics, folded by the last workgroup (a tile
    // past the live agents, so it has time to spare); this step adds to the
    // other half of the accumulators
    if (a.fold_row && blockIdx.x == gridDim.x - 1)
        fold_stats(a.acc + (kHalfLanes - a.acc_par), a.fold_row);
    // the next step's marks start from zero (K3 raises them)
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x < 2 * kMarkLanes) a.mark_wr[threadIdx.x] = 0;
    move_claim(a, block_of(a, blockIdx.x), lds);
}

// K1b (multi_prey): wolf j of cell c takes rank r among the wolves of c (eat
// keys) and eats the sheep of rank r among the sheep of c (prey keys), if the
// cell has that many.  Ranks are counted over the cell's lists; the lists of a
// cell are short at the workloads' densities (a few agents), and the count is
// quadratic in the sheep of one cell at worst.  Distinct wolves of a cell
// have distinct ranks, so no sheep is taken twice.
__device__ __forceinline__ void prey_match(const StepArgs& a, int64_t j) {
    if (j >= a.cap_w || a.sp[1].alive[j] == 0) return;
    const int64_t c = cell_of(a.sp[1].x[j], a.sp[1].y[j], a.W, a.H);
    if (c < 0) return;
    const uint64_t skey = stream_key(a.seed, a.step);
    const uint64_t my_key = agent_key(skey, j, kWolfEatKey);
    uint32_t r = 0;
    for (int32_t w = head_slot(a, a.claims[3 * c + 2]); w >= 0; w = a.blist[1][w])
        r += agent_key(skey, w, kWolfEatKey) < my_key;
    const int32_t first = head_slot(a, a.claims[3 * c + 1]);
    for (int32_t q = first; q >= 0; q = a.blist[0][q]) {
        const uint64_t kq = agent_key(skey, q, kSheepPreyKey);
        uint32_t below = 0;
        for (int32_t u = first; u >= 0; u = a.blist[0][u])
            below += agent_key(skey, u, kSheepPreyKey) < kq;
        if (below == r) {
            a.sp[0].alive[q] = 2;
            a.sp[1].e[j] += a.gain_w;
            return;
        }
    }
}

__global__ __launch_bounds__(kBlock) void k_prey_match(StepArgs a) {
    prey_match(a, int64_t(blockIdx.x) * kBlock + threadIdx.x);
}

// ------------------------------------------------------------------ K2
struct EatLds {
    uint32_t breeds[kBlockWords], gone[kBlockWords];
    uint32_t lds[2 * kThreadWaves + 1];
};

__device__ __forceinline__ void eat_breeders(const StepArgs& a, const Block& b, uint32_t epoch,
                                             EatLds& sh) {
    uint32_t *const breeds = sh.breeds, *const gone = sh.gone, *const lds = sh.lds;
    const int s = b.s;
    const int64_t cap = s ? a.cap_w : a.cap_s;
    // blocks at or past the mark hold no live agent: no breeder, every slot
    // free; they take no part in the scans (no block below them reads their
    // words), and K3 derives their free-slot prefixes from the totals
    const uint32_t mark = mark_of(a, s);
    if (b.q >= mark) {
        if (mark == 0 && b.q == 0 && threadIdx.x == 0) {
            *pick(a.d_nb, s) = 0;
            *pick(a.d_nf, s) = cap;
        }
        return;
    }
    const Species sp = species_at(pick(a.sp, s), b.base);
    const uint32_t base = uint32_t(b.base);
    breeds[threadIdx.x] = 0;
    gone[threadIdx.x] = 0;
    __syncthreads();
    const uint64_t skey = stream_key(a.seed, a.step);
    uint32_t grass_eaten = 0, sheep_eaten = 0;
    for (uint32_t w0 = 0; w0 < b.words; w0 += kOwners) {
        const uint32_t live = live_of(a, b, w0);
        if (__ballot(live != 0u) == 0) continue;   // (the wave's)
        uint32_t i[kPerThread];
        int32_t c[kPerThread], e[kPerThread];
        uint32_t eaten = 0;
#pragma unroll
        for (int k = 0; k < kPerThread; ++k) {
            const bool on = (live >> k) & 1u;
            i[k] = on ? slot_in_block(w0, k) : 0u;
            const int32_t x = sp.x[i[k]], y = sp.y[i[k]];
            e[k] = sp.e[i[k]];
            c[k] = on ? int32_t(cell_of(x, y, a.W, a.H)) : -1;
            if (a.multi && s == 0 && on && sp.alive[i[k]] == 2) eaten |= 1u << k;
        }
        uint64_t mine[kPerThread], other[kPerThread];
#pragma unroll
        for (int k = 0; k < kPerThread; ++k) {
            // sheep: the grass word and the eater's; wolves: the eater's and the prey's
            const uint64_t* cell = a.claims + 3 * int64_t(c[k] < 0 ? 0 : c[k]);
            mine[k] = cell[s ? 2 : 0];
            other[k] = cell[s ? 1 : 2];
        }
#pragma unroll
        for (int k = 0; k < kPerThread; ++k) {
            if (c[k] < 0) continue;
            if (s == 0) {
                if (mine[k] == claim_key(a, skey, base + i[k], kSheepGrassKey)) {
                    e[k] += a.gain_s;
                    sp.e[i[k]] = e[k];
                    a.ready[c[k]] = int32_t(a.step + uint32_t(a.R));
                    ++grass_eaten;
                }
                if (!a.multi && claimed(a, other[k]) &&
                    a.claims[3 * int64_t(c[k]) + 1] == claim_key(a, skey, base + i[k], kSheepPreyKey)) {
                    sp.alive[i[k]] = 2;
                    eaten |= 1u << k;
                }
            } else if (!a.multi && claimed(a, other[k]) &&
                       mine[k] == claim_key(a, skey, base + i[k], kWolfEatKey)) {
                // (multi_prey: K1b has already added the gain)
                e[k] += a.gain_w;
                sp.e[i[k]] = e[k];
            }
        }
        sheep_eaten += __popc(eaten);
#pragma unroll
        for (int k = 0; k < kPerThread; ++k) {
            if (!((live >> k) & 1u)) continue;
            if ((eaten >> k) & 1u)
                set_bit(gone, slot_in_block(w0, k));   // its slot is free for this step's births
            else if (e[k] > 0 && draw(skey, base + i[k], s ? kWolfBreed : kSheepBreed) <
                                     (s ? a.T_w : a.T_s))
                set_bit(breeds, slot_in_block(w0, k));
        }
    }
    __syncthreads();
    // breeders (compacted in slot order for K3) and the slots free for this
    // step's births (empty, or eaten this step), ranked over two chains at
    // once; a thread per bitmask word of the block
    const uint32_t w = threadIdx.x;
    const uint32_t bm = breeds[w];
    const uint32_t mask = w < b.words ? pick(a.bits, s)[b.word0 + w] : 0u;
    const uint32_t free_m = (~mask & word_in_cap(b, w, cap)) | gone[w];
    uint32_t r0, rf;
    const uint32_t total = rank_block(__popc(bm), &r0, lds);
    const uint32_t total_f = rank_block(__popc(free_m), &rf, lds + kThreadWaves);
    uint32_t excl, free_excl;
    hier_prefix2(a.status + pick(a.chain_off, s), a.status + pick(a.fchain_off, s), a.err, b.q,
                 pick(a.blocks, s), epoch, total, total_f, lds, &excl, &free_excl);
    uint32_t r = excl + r0;
    for (uint32_t m = bm; m; m &= m - 1u)
        pick(a.blist, s)[r++] = int32_t(b.base + w * 32u + (__ffs(m) - 1));
    if (threadIdx.x == 0) {
        pick(a.free_pre, s)[b.q] = int32_t(free_excl);
        if (b.q == mark - 1) {
            const int64_t past = cap - int64_t(first_tile(mark)) * kTile;
            *pick(a.d_nb, s) = int64_t(excl) + total;
            *pick(a.d_nf, s) = int64_t(free_excl) + total_f + (past > 0 ? past : 0);
        }
    }
    if (a.stats && s == 0) {
        block_add(grass_eaten, a.acc + a.acc_par, kGrassEaten, lds);
        block_add(sheep_eaten, a.acc + a.acc_par, kSheepEaten, lds);
    }
}

__global__ __launch_bounds__(kThreads) void k_eat_breeders(StepArgs a) {
    __shared__ EatLds sh;
    eat_breeders(a, block_of(a, blockIdx.x), read_epoch(a.epoch), sh);
}

// ------------------------------------------------------------------ K3
struct BreedLds {
    uint16_t list[kTile * kTilesPerBlock];
    uint32_t gone[kBlockWords], starves[kBlockWords];
    uint32_t lds[kThreadWaves + 1];
};

// At the end of a tag period each workgroup (b of n) re-arms its slice of the
// claim tables for the next step (K2, the last reader, has finished): whole
// lines, streamed.
__device__ __forceinline__ void rearm_slice(const StepArgs& a, uint32_t b, uint32_t n) {
    const int64_t words = 3 * a.G, per = (words + n - 1) / n;
    const int64_t lo = int64_t(b) * per;
    const int64_t hi = lo + per < words ? lo + per : words;
    for (int64_t w = lo + threadIdx.x; w < hi; w += kThreads) a.claims[w] = kNoClaim;
}

__device__ __forceinline__ void breed_die(const StepArgs& a, const Block& b, BreedLds& sh) {
    uint16_t* const list = sh.list;
    uint32_t *const gone = sh.gone, *const starves = sh.starves, *const lds = sh.lds;
    const int s = b.s;
    const int64_t cap = s ? a.cap_w : a.cap_s;
    const int64_t nb = *pick(a.d_nb, s), nfree = *pick(a.d_nf, s);
    if (a.stats && b.q == pick(a.blocks, s) - 1 && threadIdx.x == 0)
        a.stats[s ? kBirthsW : kBirthsS] = nfree < nb ? nfree : nb;
    // the block's free-slot prefix: from K2's scan below the mark; past it every
    // slot of every block is free
    const uint32_t mark = mark_of(a, s);
    int64_t pre;
    if (b.q < mark) {
        pre = pick(a.free_pre, s)[b.q];
    } else {
        const int64_t first = int64_t(first_tile(mark)) * kTile;
        pre = nfree - (cap - first > 0 ? cap - first : 0) + (b.base - first);
        // with no live agent and no birth (its free slots rank past the
        // breeders) there is nothing to do
        if (pre >= nb) return;
    }
    const Species sp = pick(a.sp, s), here = species_at(sp, b.base);
    gone[threadIdx.x] = 0;
    starves[threadIdx.x] = 0;
    __syncthreads();
    // eaten sheep become free slots, starving agents die
    uint32_t starved = 0;
    for (uint32_t w0 = 0; w0 < b.words && b.q < mark; w0 += kOwners) {
        const uint32_t live = live_of(a, b, w0);
        if (__ballot(live != 0u) == 0) continue;   // (the wave's)
        uint32_t i[kPerThread];
        int32_t al[kPerThread], e[kPerThread];
#pragma unroll
        for (int k = 0; k < kPerThread; ++k) {
            i[k] = (live >> k) & 1u ? slot_in_block(w0, k) : 0u;
            al[k] = here.alive[i[k]];
            e[k] = here.e[i[k]];
        }
#pragma unroll
        for (int k = 0; k < kPerThread; ++k) {
            if (!((live >> k) & 1u)) continue;
            if (al[k] == 2) {               // eaten: a free slot for this step's births
                set_bit(gone, slot_in_block(w0, k));
                here.alive[i[k]] = 0;
            } else if (e[k] < 0) {
                // a breeder's energy stays positive, so no slot read by a child dies here
                set_bit(starves, slot_in_block(w0, k));
                here.alive[i[k]] = 0;
                ++starved;
            }
        }
    }
    __syncthreads();
    const uint32_t w = threadIdx.x;
    const uint32_t mask = w < b.words ? pick(a.bits, s)[b.word0 + w] : 0u;   // live at K1
    const uint32_t free_m = (~mask & word_in_cap(b, w, cap)) | gone[w];
    // (the same free slots K2 ranked: its chain gave this block's prefix)
    uint32_t r0;
    const uint32_t total = rank_block(__popc(free_m), &r0, lds);
    const uint32_t excl = uint32_t(pre);
    const int64_t room = nb - int64_t(excl);
    const uint32_t births = room <= 0 ? 0u : (room < int64_t(total) ? uint32_t(room) : total);
    // this word's free slots of block rank < births receive children; they are
    // the block's first ones, so their rank is their place in the list
    uint32_t born_m = 0, r = r0;
    for (uint32_t m = free_m; m && r < births; m &= m - 1u, ++r) {
        born_m |= m & (0u - m);
        list[r] = uint16_t(w * 32u + (__ffs(m) - 1));
    }
    const uint32_t live_m = (mask & ~gone[w] & ~starves[w]) | born_m;
    if (w < b.words && live_m != mask) pick(a.bits, s)[b.word0 + w] = live_m;
    // the next step's mark: past the last block left with a live agent
    if (__syncthreads_or(live_m != 0u) && threadIdx.x == 0)
        atomicMax(reinterpret_cast<unsigned long long*>(a.mark_wr + s * kMarkLanes +
                                                        (b.q & (kMarkLanes - 1))),
                  (unsigned long long)(b.q + 1));
    // the children, spread over the workgroup
    for (uint32_t j = threadIdx.x; j < births; j += kThreads) {
        const int64_t ci = b.base + list[j], p = pick(a.blist, s)[excl + j];
        const int32_t px = sp.x[p], py = sp.y[p], pe = sp.e[p];
        const int32_t ec = pe >> 1;
        sp.x[ci] = px;
        sp.y[ci] = py;
        sp.e[ci] = ec;
        sp.e[p] = pe - ec;
        sp.alive[ci] = 1;
    }
    if (a.stats) block_add(starved, a.acc + a.acc_par, s ? kStarvedW : kStarvedS, lds);
}

__global__ __launch_bounds__(kThreads) void k_breed_die(StepArgs a) {
    __shared__ BreedLds sh;
    if (a.rearm) rearm_slice(a, blockIdx.x, gridDim.x);
    breed_die(a, block_of(a, blockIdx.x), sh);
}

// ------------------------------------------------------------------ call edges
// Bitmask word k of the live slots.  A caller's 2, the mark of an eaten sheep
// within a step, becomes 1.
__device__ __forceinline__ uint32_t live_word(int32_t* alive, int64_t k, int64_t cap) {
    int32_t* al = alive + k * 32;
    uint32_t m = 0, twos = 0;
    if (k * 32 + 32 <= cap) {
        int4 v[8];
        __builtin_memcpy(v, al, sizeof v);      // (4-byte alignment is enough)
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            m |= uint32_t(v[q].x != 0) << (4 * q) | uint32_t(v[q].y != 0) << (4 * q + 1) |
                 uint32_t(v[q].z != 0) << (4 * q + 2) | uint32_t(v[q].w != 0) << (4 * q + 3);
            twos |= uint32_t(v[q].x == 2) << (4 * q) | uint32_t(v[q].y == 2) << (4 * q + 1) |
                    uint32_t(v[q].z == 2) << (4 * q + 2) | uint32_t(v[q].w == 2) << (4 * q + 3);
        }
    } else {
        for (int b = 0; b < 32 && k * 32 + b < cap; ++b) {
            m |= uint32_t(al[b] != 0) << b;
            twos |= uint32_t(al[b] == 2) << b;
        }
    }
    for (; twos; twos &= twos - 1u) al[__ffs(twos) - 1] = 1;
    return m;
}

// Start of a call: grass countdowns -> ready steps, live bitmasks from alive,
// every claim word re-armed.  One thread per bitmask word (and cell).
__global__ __launch_bounds__(kBlock) void k_call_begin(StepArgs a, int64_t G, int64_t words_s,
                                                       int64_t words_w) {
    const int64_t k = int64_t(blockIdx.x) * kBlock + threadIdx.x;
    // the first step visits every block
    if (k < 2 * kMarkLanes) a.mark_rd[k] = a.blocks[k / kMarkLanes];
    if (k < G) {
        a.ready[k] = int32_t(a.step + uint32_t(a.ready[k]));
        a.claims[3 * k] = kNoClaim;
        a.claims[3 * k + 1] = kNoClaim;
        a.claims[3 * k + 2] = kNoClaim;
    }
    if (k < words_s) a.bits[0][k] = live_word(a.sp[0].alive, k, a.cap_s);
    if (k < words_w) a.bits[1][k] = live_word(a.sp[1].alive, k, a.cap_w);
}

// End of a call: ready steps -> countdowns at step `end`.
__global__ __launch_bounds__(kBlock) void k_call_end(int32_t* grass, int64_t G, uint32_t end) {
    const int64_t c = int64_t(blockIdx.x) * kBlock + threadIdx.x;
    if (c < G) {
        const int32_t d = int32_t(uint32_t(grass[c]) - end);
        grass[c] = d > 0 ? d : 0;
    }
}

// The last step's fold (every other step's is done by the next step's K1).
__global__ __launch_bounds__(kBlock) void k_fold_stats(int64_t* acc, int64_t* stats) {
    fold_stats(acc, stats);
}

// Slot bits, first tag and steps of a tag period for slots below max_cap.
struct Tags {
    uint32_t sb, top, period;
};

__host__ __device__ __forceinline__ Tags tags_for(int64_t max_cap) {
    uint32_t sb = 1;
    while (sb < 31 && (int64_t(1) << sb) < max_cap) ++sb;
    const uint32_t tag_bits = 32 - sb < kTagBits ? 32 - sb : kTagBits;
    const uint32_t t_max = (1u << tag_bits) - 1;
    return Tags{sb, t_max > 1 ? t_max - 1 : 0u, t_max > 1 ? t_max - 1 : 1u};
}

// ------------------------------------------------------------------ batches
// Large models of a batch (`wide` models), all of them side by side: the launches
// above with the workgroups shared out among the models.  96 models of 32^2
// to 1024^2 cells x 40 steps take 10.4 ms, bound as the one-model launches are
// by the atomics and the claim lines of 1.7 M agents (34.5 ms by teams of four
// workgroups, whose chain of dependent accesses per agent the largest model's
// team went through alone).  A model's
// arguments are built on the device, from its descriptor, in its share of the
// workspace: the breeder lists in one half of it; the arguments, marks, totals,
// scan words and live bitmasks in the other.
struct WideLayout {
    int64_t status, free_pre, bits[2], end;   // byte offsets
};

struct WideModel {
    StepArgs a;                           // what does not change (no pointers)
    WideLayout at;
    Tags tags;
    int64_t cell_off, slot_off[2];
    uint32_t step0;
    int32_t index;                        // of the model
    int32_t n;                            // steps of this call
    unsigned long long updates;
    uint64_t marks[2][2][kMarkLanes];
    int64_t nb[2], nf[2];
};

__host__ __device__ __forceinline__ WideLayout wide_layout(uint32_t tiles_s, uint32_t tiles_w) {
    const uint32_t b0 = blocks_of(tiles_s), b1 = blocks_of(tiles_w);
    WideLayout l;
    l.status = (int64_t(sizeof(WideModel)) + 63) / 64 * 64;
    l.free_pre = l.status + 16 * (chain_words(b0) + chain_words(b1));
    l.bits[0] = l.free_pre + 4 * (int64_t(b0) + b1);
    l.bits[1] = l.bits[0] + 4 * int64_t(tiles_s) * kOwners;
    l.end = l.bits[1] + 4 * int64_t(tiles_w) * kOwners;
    return l;
}

__device__ __forceinline__ WideModel* wide_model(const WideArgs& w, uint32_t k) {
    return reinterpret_cast<WideModel*>(w.shares + (2 * int64_t(k) + 1) * w.share);
}

// One workgroup per model that may be taken: the k-th taken one gets the k-th
// pair of shares, its arguments, its counters and scan words cleared there.
__global__ __launch_bounds__(kBlock) void k_wide_begin(WideArgs w) {
    const int32_t y = int32_t(blockIdx.x);
    const auto taken = [&](int32_t i) { return i < w.n_team || w.taken[i] != 0; };
    int32_t k = 0;
    for (int32_t i0 = 0; i0 < y; i0 += kBlock) {
        const int32_t i = i0 + int32_t(threadIdx.x);
        k += __syncthreads_count(i < y && taken(i));
    }
    if (y == w.n - 1 && threadIdx.x == 0) *w.count = uint32_t(k + (taken(y) ? 1 : 0));
    if (!taken(y)) return;
    WideModel* const m = wide_model(w, uint32_t(k));
    const int32_t index = w.order[y];
    const abm_model_desc& d = w.models[index];
    const bool links = w.link_s && w.link_w;
    // as a workgroup's model: refused if it does not fit the lists
    const bool bad = d.cap_s + d.cap_w > 2 * w.max_cap || (d.multi_prey && !links);
    const int32_t left = d.steps_target - d.step;
    const int32_t n = bad || left <= 0 ? 0 : (left < w.max_steps ? left : w.max_steps);
    if (n == 0) {
        if (threadIdx.x == 0) {
            m->n = 0;
            if (bad) st_agent(w.err, 1ull);
        }
        return;
    }
    const uint32_t tiles_s = uint32_t((d.cap_s + kTile - 1) / kTile);
    const uint32_t tiles_w = uint32_t((d.cap_w + kTile - 1) / kTile);
    const WideLayout l = wide_layout(tiles_s, tiles_w);
    char* const base = reinterpret_cast<char*>(m);
    for (int64_t i = threadIdx.x; i < (l.free_pre - l.status) / 8; i += kBlock)
        reinterpret_cast<uint64_t*>(base + l.status)[i] = 0;   // (no step's epoch)
    if (threadIdx.x != 0) return;
    StepArgs a = {};
    a.W = d.W;
    a.H = d.H;
    a.R = d.R;
    a.gain_s = d.gain_s;
    a.gain_w = d.gain_w;
    a.T_s = d.T_s;
    a.T_w = d.T_w;
    a.seed = d.seed;
    a.cap_s = d.cap_s;
    a.cap_w = d.cap_w;
    a.G = int64_t(d.W) * d.H;
    a.multi = d.multi_prey != 0;
    a.batch = 1;
    a.tiles[0] = tiles_s;
    a.tiles[1] = tiles_w;
    a.blocks[0] = blocks_of(tiles_s);
    a.blocks[1] = blocks_of(tiles_w);
    const int64_t cw0 = chain_words(a.blocks[0]), cw1 = chain_words(a.blocks[1]);
    a.chain_off[1] = uint32_t(cw0);
    a.fchain_off[0] = uint32_t(cw0 + cw1);
    a.fchain_off[1] = uint32_t(2 * cw0 + cw1);
    for (int s = 0; s < 2; ++s)
        for (int q = 0; q < kMarkLanes; ++q) m->marks[0][s][q] = a.blocks[s];
    m->tags = tags_for(d.cap_s > d.cap_w ? d.cap_s : d.cap_w);
    a.sb = m->tags.sb;
    a.tag_mask = ~uint64_t(0) << (32 + a.sb);
    m->a = a;
    m->at = l;
    m->cell_off = d.cell_off;
    m->slot_off[0] = d.sheep_off;
    m->slot_off[1] = d.wolf_off;
    m->step0 = uint32_t(d.step);
    m->index = index;
    m->n = n;
    atomicMax(w.count + 1, uint32_t(n));
    m->updates = 0;
}

// The model's arguments at step k of the call.
__device__ __forceinline__ StepArgs wide_step(const WideArgs& w, WideModel* m, int32_t k) {
    StepArgs a = m->a;
    // (pointers made of the launch's arguments are known to be global; read
    // from memory they could point anywhere, and every access would be a flat one)
    char* const base = reinterpret_cast<char*>(m);
    a.ready = w.ready + m->cell_off;
    a.claims = w.claims + 3 * m->cell_off;
    a.sp[0] = Species{w.sheep.x + m->slot_off[0], w.sheep.y + m->slot_off[0],
                      w.sheep.e + m->slot_off[0], w.sheep.alive + m->slot_off[0]};
    a.sp[1] = Species{w.wolves.x + m->slot_off[1], w.wolves.y + m->slot_off[1],
                      w.wolves.e + m->slot_off[1], w.wolves.alive + m->slot_off[1]};
    a.bits[0] = reinterpret_cast<uint32_t*>(base + m->at.bits[0]);
    a.bits[1] = reinterpret_cast<uint32_t*>(base + m->at.bits[1]);
    a.status = reinterpret_cast<uint64_t*>(base + m->at.status);
    a.err = w.err;
    a.updates = &m->updates;
    a.free_pre[0] = reinterpret_cast<int32_t*>(base + m->at.free_pre);
    a.free_pre[1] = a.free_pre[0] + a.blocks[0];
    a.blist[0] = reinterpret_cast<int32_t*>(base - w.share);
    a.blist[1] = a.blist[0] + a.cap_s;
    for (int s = 0; s < 2; ++s) {
        a.d_nb[s] = &m->nb[s];
        a.d_nf[s] = &m->nf[s];
    }
    const uint32_t phase = uint32_t(k) % m->tags.period;
    a.step = m->step0 + uint32_t(k);
    a.tag_hi = uint64_t(m->tags.top - phase) << (32 + m->tags.sb);
    // (the tables are all-ones between runs)
    a.rearm = phase == m->tags.period - 1 || k + 1 == m->n;
    a.mark_rd = &m->marks[k & 1][0][0];
    a.mark_wr = &m->marks[(k + 1) & 1][0][0];
    return a;
}

// The model of this workgroup (null: none), and the workgroup's number among the
// `per` of the model.
struct WideGroup {
    WideModel* m;
    uint32_t x, per;
};

// The workgroups of the launch are divided among the models taken, whose number
// only the device knows: a model has 8 times an odd number of consecutive ones.
// Consecutive workgroups go to the eight XCDs in turn, and on an XCD to its 32
// CUs in turn; with an even share of each XCD the low blocks of the models,
// where the live agents are, would meet on the same CUs (200 models of 64^2 to
// 500^2 cells x 20 steps: 3.1 ms with 24 workgroups a model, 4.0 with 32, 3.4 with 48;
// 96 of 32^2 to 1024^2: 6.0, 6.6, 6.1).  Many models take few each (200 of 300^2
// to 430^2: 10.0 ms with 8, 11.6 with 48).  No model takes more than kWideShare,
// though one alone would gain (1000^2: 1.69 ms with 48, 0.81 with 256): a
// workgroup with several blocks waits for the later ones of its model, so an XCD
// has to hold a model's seven workgroups at once, beside what the launches of
// other streams hold.
constexpr uint32_t kWideShare = 56;

__device__ __forceinline__ WideGroup wide_group(const WideArgs& w, int32_t step) {
    const uint32_t n = w.count[0];
    // (a launch past every model's last step costs one load of each workgroup)
    if (uint32_t(step) >= w.count[1]) return WideGroup{nullptr, 0, 1};
    uint32_t per = gridDim.x / n < kWideShare ? gridDim.x / n : kWideShare;
    per = 8 * (((per / 8 > 1 ? per / 8 : 1) - 1) | 1);
    const uint32_t k = blockIdx.x / per;
    return WideGroup{k < n ? wide_model(w, k) : nullptr, blockIdx.x - k * per, per};
}

__global__ __launch_bounds__(kBlock) void k_wide_bits(WideArgs w) {
    const WideGroup g = wide_group(w, 0);
    if (!g.m || g.m->n == 0) return;
    const StepArgs a = wide_step(w, g.m, 0);
    const int64_t words_s = int64_t(a.tiles[0]) * kOwners, words_w = int64_t(a.tiles[1]) * kOwners;
    for (int64_t k = int64_t(g.x) * kBlock + threadIdx.x; k < words_s || k < words_w;
         k += int64_t(g.per) * kBlock) {
        if (k < words_s) a.bits[0][k] = live_word(a.sp[0].alive, k, a.cap_s);
        if (k < words_w) a.bits[1][k] = live_word(a.sp[1].alive, k, a.cap_w);
    }
}

// Runs body(arguments, block) over this workgroup's blocks of its model.  A
// model's workgroups are consecutive, so the smallest unfinished block of its
// scans is always that of a resident one.
template <class F>
__device__ __forceinline__ void wide_blocks(const WideGroup& g, const StepArgs& a, F body) {
    const uint32_t n = a.blocks[0] + a.blocks[1];
    for (uint32_t i = g.x; i < n; i += g.per) {
        if (i != g.x) __syncthreads();
        body(block_of(a, i));
    }
}

__global__ __launch_bounds__(kThreads) void k_wide_move(WideArgs w, int32_t k) {
    __shared__ uint32_t lds[kThreadWaves];
    const WideGroup g = wide_group(w, k);
    if (!g.m || k >= g.m->n) return;
    const StepArgs a = wide_step(w, g.m, k);
    if (g.x == 0 && threadIdx.x < 2 * kMarkLanes) a.mark_wr[threadIdx.x] = 0;
    wide_blocks(g, a, [&](const Block& b) { move_claim(a, b, lds); });
}

__global__ __launch_bounds__(kBlock) void k_wide_match(WideArgs w, int32_t k) {
    const WideGroup g = wide_group(w, k);
    if (!g.m || k >= g.m->n || !g.m->a.multi) return;
    const StepArgs a = wide_step(w, g.m, k);
    for (int64_t j = int64_t(g.x) * kBlock + threadIdx.x; j < a.cap_w; j += int64_t(g.per) * kBlock)
        prey_match(a, j);
}

__global__ __launch_bounds__(kThreads) void k_wide_eat(WideArgs w, int32_t k) {
    __shared__ EatLds sh;
    const WideGroup g = wide_group(w, k);
    if (!g.m || k >= g.m->n) return;
    const StepArgs a = wide_step(w, g.m, k);
    wide_blocks(g, a, [&](const Block& b) { eat_breeders(a, b, uint32_t(k) + 1u, sh); });
}

__global__ __launch_bounds__(kThreads) void k_wide_breed(WideArgs w, int32_t k) {
    __shared__ BreedLds sh;
    const WideGroup g = wide_group(w, k);
    if (!g.m || k >= g.m->n) return;
    const StepArgs a = wide_step(w, g.m, k);
    if (a.rearm) rearm_slice(a, g.x, g.per);
    wide_blocks(g, a, [&](const Block& b) { breed_die(a, b, sh); });
}

__global__ __launch_bounds__(64) void k_wide_end(WideArgs w) {
    if (blockIdx.x >= *w.count || threadIdx.x != 0) return;
    const WideModel* const m = wide_model(w, blockIdx.x);
    if (m->n == 0) return;
    abm_model_desc& d = w.models[m->index];
    d.step += m->n;
    d.updates += int64_t(m->updates);
}

int check_params(const abm_predation_params* p) {
    if (!p) return fail(ABM_E_INVALID, "params are NULL");
    if (p->W < 1 || p->H < 1 || int64_t(p->W) * p->H > kMaxIndex)
        return fail(ABM_E_INVALID, "grid must satisfy W, H >= 1 and W*H < 2^31");
    if (p->R < 1) return fail(ABM_E_INVALID, "R must be >= 1");
    if (p->gain_s < 0 || p->gain_w < 0 || p->gain_s > (1 << 29) || p->gain_w > (1 << 29))
        return fail(ABM_E_INVALID, "gains must be in [0, 2^29]");
    if (p->cap_s < 1 || p->cap_w < 1 || p->cap_s > kMaxIndex || p->cap_w > kMaxIndex)
        return fail(ABM_E_INVALID, "capacities must be in [1, 2^31)");
    if (p->cap_s + p->cap_w > kMaxIndex)
        return fail(ABM_E_INVALID, "cap_s + cap_w must be below 2^31");
    if (p->n_s0 < 0 || p->n_w0 < 0 || p->n_s0 > p->cap_s || p->n_w0 > p->cap_w)
        return fail(ABM_E_INVALID, "initial counts must be in [0, capacity]");
    if (p->multi_prey != 0 && p->multi_prey != 1)
        return fail(ABM_E_INVALID, "multi_prey must be 0 or 1");
    return ABM_OK;
}

int check_state(const abm_predation_state* s) {
    if (!s) return fail(ABM_E_INVALID, "state is NULL");
    if (!s->grass || !s->claims) return fail(ABM_E_INVALID, "grass or claims is NULL");
    const abm_species* sp[2] = {&s->sheep, &s->wolves};
    for (int k = 0; k < 2; ++k)
        if (!sp[k]->x || !sp[k]->y || !sp[k]->e || !sp[k]->alive)
            return fail(ABM_E_INVALID, "species array is NULL");
    return ABM_OK;
}

Species species_of(const abm_species& s) { return Species{s.x, s.y, s.e, s.alive}; }

}  // namespace
}  // namespace abm

namespace abm {

// Workgroups of a launch, unless eight a model are more.  (A launch that finds
// nothing to do costs their dispatch: 2.3 us; with 3072, 3.  96 models of 32^2 to
// 1024^2 cells x 40 steps: 10.4 ms, and 10.5 with 3072.)
constexpr int64_t kWideGroups = 1920;

bool wide_fits(int64_t max_cap) {
    // (a descriptor may split the 2 max_cap slots otherwise: a tile more at most)
    const uint32_t tiles = uint32_t(tiles_for(max_cap, kTile)) + 1;
    return wide_layout(tiles, tiles).end <= 8 * max_cap;
}

int launch_wide(const WideArgs& w, hipStream_t st) {
    int64_t groups = int64_t(w.n) * kWideShare;
    if (groups > kWideGroups) groups = kWideGroups > 8 * int64_t(w.n) ? kWideGroups : 8 * int64_t(w.n);
    const dim3 grid{uint32_t(groups)}, block(kThreads);
    hipLaunchKernelGGL(k_wide_begin, dim3(uint32_t(w.n)), dim3(kBlock), 0, st, w);
    hipLaunchKernelGGL(k_wide_bits, grid, dim3(kBlock), 0, st, w);
    for (int32_t k = 0; k < w.max_steps; ++k) {
        hipLaunchKernelGGL(k_wide_move, grid, block, 0, st, w, k);
        if (w.link_s && w.link_w)
            hipLaunchKernelGGL(k_wide_match, grid, dim3(kBlock), 0, st, w, k);
        hipLaunchKernelGGL(k_wide_eat, grid, block, 0, st, w, k);
        hipLaunchKernelGGL(k_wide_breed, grid, block, 0, st, w, k);
    }
    hipLaunchKernelGGL(k_wide_end, dim3(uint32_t(w.n)), dim3(64), 0, st, w);
    return launch_status("predation_run_batched");
}

}  // namespace abm

using namespace abm;

extern "C" int abm_predation_init(const abm_predation_params* p, abm_predation_state* s,
                                  void* stream) {
    int rc = check_params(p);
    if (rc != ABM_OK) return rc;
    rc = check_state(s);
    if (rc != ABM_OK) return rc;
    rc = check_device();
    if (rc != ABM_OK) return rc;
    InitArgs a;
    a.W = p->W;
    a.H = p->H;
    a.R = p->R;
    a.gain_s = p->gain_s;
    a.gain_w = p->gain_w;
    a.seed = p->seed;
    a.cap_s = p->cap_s;
    a.cap_w = p->cap_w;
    a.n_s0 = p->n_s0;
    a.n_w0 = p->n_w0;
    a.G = int64_t(p->W) * p->H;
    a.grass = s->grass;
    a.sp[0] = species_of(s->sheep);
    a.sp[1] = species_of(s->wolves);
    a.claims = s->claims;
    int64_t m = a.G;
    if (a.cap_s > m) m = a.cap_s;
    if (a.cap_w > m) m = a.cap_w;
    hipLaunchKernelGGL(k_init, dim3(tiles_for(m, kBlock)), dim3(kBlock), 0, as_stream(stream), a);
    rc = launch_status("predation_init");
    if (rc == ABM_OK) s->step = 0;
    return rc;
}

extern "C" int abm_predation_step(const abm_predation_params* p, abm_predation_state* s,
                                  int32_t n_steps, void* ws, size_t ws_bytes, void* stream) {
    int rc = check_params(p);
    if (rc != ABM_OK) return rc;
    rc = check_state(s);
    if (rc != ABM_OK) return rc;
    if (n_steps < 0) return fail(ABM_E_INVALID, "n_steps must be >= 0");
    rc = check_device();
    if (rc != ABM_OK) return rc;
    const int64_t cap = p->cap_s > p->cap_w ? p->cap_s : p->cap_w;
    rc = check_ws(ws, ws_bytes, cap);
    if (rc != ABM_OK) return rc;
    if (n_steps == 0) return ABM_OK;
    Workspace w = carve(ws, cap);
    hipStream_t st = as_stream(stream);
    bool taken = false;
    rc = launch_small_predation(p, s, n_steps, w, st, &taken);
    if (taken) {
        if (rc == ABM_OK) s->step += uint32_t(n_steps);
        return rc;
    }
    const int64_t G = int64_t(p->W) * p->H;

    StepArgs a;
    a.W = p->W;
    a.H = p->H;
    a.R = p->R;
    a.gain_s = p->gain_s;
    a.gain_w = p->gain_w;
    a.T_s = p->T_s;
    a.T_w = p->T_w;
    a.seed = p->seed;
    a.cap_s = p->cap_s;
    a.cap_w = p->cap_w;
    a.ready = s->grass;
    a.sp[0] = species_of(s->sheep);
    a.sp[1] = species_of(s->wolves);
    a.bits[0] = w.bits_a;
    a.bits[1] = w.bits_b;
    a.G = G;
    a.claims = s->claims;
    a.status = w.status;
    a.err = w.status - 1;
    a.updates = nullptr;
    a.acc = w.acc;
    a.blist[0] = w.list_a;
    a.blist[1] = w.list_b;
    a.d_nb[0] = reinterpret_cast<int64_t*>(w.hdr + kHdrCountA);
    a.d_nb[1] = reinterpret_cast<int64_t*>(w.hdr + kHdrCountB);
    a.d_nf[0] = reinterpret_cast<int64_t*>(w.hdr + kHdrFreeA);
    a.d_nf[1] = reinterpret_cast<int64_t*>(w.hdr + kHdrFreeB);
    a.tiles[0] = static_cast<uint32_t>(tiles_for(p->cap_s, kTile));
    a.tiles[1] = static_cast<uint32_t>(tiles_for(p->cap_w, kTile));
    a.blocks[0] = blocks_of(a.tiles[0]);
    a.blocks[1] = blocks_of(a.tiles[1]);
    a.turn = a.blocks[0] + a.blocks[1] <= 2048 ? 3 : 0;
    // status words: the breeder chains of both species, then their free-slot
    // chains, then the per-block free prefixes (int32) K2 leaves for K3; the
    // area is sized for 512-slot tiles, four times the chains of 2048-slot tiles
    const int64_t cw0 = chain_words(a.blocks[0]), cw1 = chain_words(a.blocks[1]);
    a.chain_off[0] = 0;
    a.chain_off[1] = static_cast<uint32_t>(cw0);
    a.fchain_off[0] = static_cast<uint32_t>(cw0 + cw1);
    a.fchain_off[1] = static_cast<uint32_t>(2 * cw0 + cw1);
    const int64_t pre_words = 2 * (cw0 + cw1) + (int64_t(a.blocks[0]) + a.blocks[1] + 1) / 2;
    if (pre_words > status_words(p->cap_s > p->cap_w ? p->cap_s : p->cap_w))
        return fail(ABM_E_WORKSPACE, "predation_step: scan state does not fit the workspace");
    a.free_pre[0] = reinterpret_cast<int32_t*>(w.status + 2 * (cw0 + cw1));
    a.free_pre[1] = a.free_pre[0] + a.blocks[0];
    a.multi = p->multi_prey;
    a.batch = 0;
    a.step = s->step;
    a.stats = nullptr;
    a.acc_par = 0;
    a.fold_row = nullptr;
    a.mark_rd = w.hdr + kHdrMark;
    a.mark_wr = w.hdr + kHdrMark + 2 * kMarkLanes;
    // claim keys (claim_key): slots below 2^sb, a tag of up to kTagBits bits
    // sb + 32 bits up; a period of steps uses the tags t_max - 1 down to 1 (tag
    // 0 every step when only one tag bit is left), and its last step re-arms
    // the table.  Short periods re-arm often enough to cost little (one
    // streamed table per 14 steps) and keep every multi-step call crossing them.
    const Tags tags = tags_for(p->cap_s > p->cap_w ? p->cap_s : p->cap_w);
    a.sb = tags.sb;
    a.tag_mask = ~uint64_t(0) << (32 + tags.sb);

    const int64_t words_s = int64_t(a.tiles[0]) * kOwners, words_w = int64_t(a.tiles[1]) * kOwners;
    int64_t edge = G > words_s ? G : words_s;
    if (words_w > edge) edge = words_w;
    const dim3 grid(a.blocks[0] + a.blocks[1]), block(kThreads);
    // grass to ready steps, live bitmasks from alive, claim tables re-armed
    // (whatever the caller did to the state between calls)
    hipLaunchKernelGGL(k_call_begin, dim3(static_cast<uint32_t>(tiles_for(edge, kBlock))),
                       dim3(kBlock), 0, st, a, G, words_s, words_w);
    hipLaunchKernelGGL(k_fill64, dim3(tiles_for(kAccWords, kBlock)), dim3(kBlock), 0, st, w.acc,
                       kAccWords, int64_t(0));
    if (s->stats)
        hipLaunchKernelGGL(k_fill64, dim3(tiles_for(8 * int64_t(n_steps), kBlock)), dim3(kBlock),
                           0, st, s->stats, 8 * int64_t(n_steps), int64_t(0));
    for (int32_t k = 0; k < n_steps; ++k) {
        a.step = s->step + uint32_t(k);
        a.stats = s->stats ? s->stats + 8 * int64_t(k) : nullptr;
        a.acc_par = (k & 1) ? kHalfLanes : 0;
        a.mark_rd = w.hdr + kHdrMark + 2 * kMarkLanes * (k & 1);
        a.mark_wr = w.hdr + kHdrMark + 2 * kMarkLanes * ((k + 1) & 1);
        a.fold_row = s->stats && k > 0 ? s->stats + 8 * int64_t(k - 1) : nullptr;
        const uint32_t phase = uint32_t(k) % tags.period;
        a.tag_hi = uint64_t(tags.top - phase) << (32 + tags.sb);
        a.rearm = phase == tags.period - 1;
        hipLaunchKernelGGL(k_move_claim, grid, block, 0, st, a);
        if (a.multi)
            hipLaunchKernelGGL(k_prey_match, dim3(static_cast<uint32_t>(tiles_for(p->cap_w, kBlock))),
                               dim3(kBlock), 0, st, a);
        rc = next_epoch(w, st, &a.epoch);
        if (rc != ABM_OK) return rc;
        hipLaunchKernelGGL(k_eat_breeders, grid, block, 0, st, a);
        hipLaunchKernelGGL(k_breed_die, grid, block, 0, st, a);
    }
    if (s->stats)
        hipLaunchKernelGGL(k_fold_stats, dim3(1), dim3(kBlock), 0, st, w.acc + a.acc_par, a.stats);
    hipLaunchKernelGGL(k_call_end, dim3(static_cast<uint32_t>(tiles_for(G, kBlock))), dim3(kBlock),
                       0, st, s->grass, G, s->step + uint32_t(n_steps));
    rc = launch_status("predation_step");
    if (rc == ABM_OK) s->step += uint32_t(n_steps);
    return rc;
}
