// lob.hip -- abm_lob_init / abm_lob_step: noisy traders on many limit order
// books, every book matched at once each step (Sec. 5.3, Fig. 5; the paper
// vectorises the matching over books, Table 4).
//
// One workgroup owns one book for a whole call, with the book's order slots
// (price, qty, time, live bit) in LDS, and beside them each side's live orders
// as a list of 64-bit priority keys (price, then time, then slot), which is
// built once per call and kept in order from step to step.  A step:
//   expiry    orders placed E or more steps ago leave the list;
//   orders    trader k orders when its draw is below T_order; the new orders,
//             in trader order, take the lowest free slots (the j-th new order
//             the j-th lowest free slot, as add_agents);
//   merge     the new orders go into their side's list: every order moves to
//             the number of orders before it;
//   matching  V = max over buys r of min(CB_r, CS(p_r)), CB and CS the
//             cumulative shares along the lists; only the top of the book can
//             match, so one wave reads the first 64 orders of each side;
//   fills     an order fills the part of its share range below V: filled
//             orders are removed, partly filled ones keep the rest; the new
//             last price is the floor of the mean of the buy and sell prices
//             covering share V.
// Draws are keyed on (seed + book, step, trader, purpose).
#include <hip/hip_runtime.h>

#include "abm.h"
#include "common.hpp"
#include "rng.hpp"
#include "wave.hpp"

namespace abm {
namespace {

constexpr int kBlock = 512;
constexpr int kWaves = kBlock / 64;
constexpr int kSideWaves = kWaves / 2;   // waves per side of the book
constexpr int kMaxCap = 1024;
constexpr int kMaxTraders = 1024;
constexpr int32_t kMaxPrice = (1 << 24) - 1;

enum LobPurpose : uint32_t { kLobOrder = 0x40, kLobSide = 0x41, kLobPrice = 0x42, kLobQty = 0x43 };
enum LobCol : int {
    kBuys = 0, kSells, kPlaced, kDropped, kExpired, kVolume, kFilled, kPrice, kCols
};

struct LobArgs {
    int32_t cap, traders;
    uint32_t T_order;
    int32_t spread, max_qty, expiry, price0;
    uint32_t seed;
    int32_t *side, *price, *qty, *time, *alive, *last_price;
    int64_t* stats;
    int32_t n_books;
    uint32_t step0;
    int32_t n_steps;
};

// LDS of a book with C slots, T traders and at most M new orders a step, in
// this order: two buffers of priority keys (the lists of a step and of the
// next), the new orders' keys, the traders' draws of two steps, each side's
// new orders' (price, index) words, each slot's price, shares and time, one
// word per list position (cum), a histogram over the new orders, the live bits
// of the slots, the free slots of a step, a byte per slot.  A list buffer
// holds the buys' keys from its start and the sells' from its end, each in
// priority order (no more than C orders are live); so do cum, the new keys and
// the histogram.
constexpr int kBitWords = kMaxCap / 32;
constexpr int kRows = kMaxCap / 64;
constexpr int kTraderChunks = kMaxTraders / 64;
constexpr int kListChunks = kMaxCap / 64;

__host__ __device__ __forceinline__ int32_t new_max(int32_t cap, int32_t traders) {
    return traders < cap ? traders : cap;
}

// Words for a side's new prices: at most kWordRanks of them, padded to whole
// groups of eight.
constexpr int kWordRanks = 256;
__host__ __device__ __forceinline__ int32_t word_room(int32_t M) {
    return ((M < kWordRanks ? M : kWordRanks) + 7) & ~7;
}

size_t lob_lds_bytes(int32_t C, int32_t T) {
    const int32_t M = new_max(C, T);
    return size_t(8) * (2 * C + M + 2 * T) +
           size_t(4) * (3 * C + (C + 2) + 2 * word_room(M) + (M + 2) + kBitWords + 4) +
           size_t(2 * M + C);
}

// Priority key of a live order, smaller is matched first within a side: side
// (bit 63), price (24 bits, reversed for buys), time (24), slot (15).
constexpr uint64_t kSellBit = uint64_t(1) << 63;

__device__ __forceinline__ uint64_t priority_key(bool sell, int32_t price, int32_t time,
                                                 int32_t slot) {
    const uint64_t p = uint64_t(uint32_t(sell ? price : kMaxPrice - price) & 0xFFFFFFu);
    return (sell ? kSellBit : 0ull) | (p << 39) | (uint64_t(uint32_t(time) & 0xFFFFFFu) << 15) |
           uint64_t(slot);
}

__device__ __forceinline__ int32_t slot_of(uint64_t key) { return int32_t(key & 0x7FFFu); }
__device__ __forceinline__ uint32_t price_of(uint64_t key) { return uint32_t(key >> 39) & 0xFFFFFFu; }

// i, or -i for neg = -1 (two full-rate operations).
__device__ __forceinline__ int32_t signed_pos(int32_t i, int32_t neg) { return (i ^ neg) - neg; }

// What a step's matching leaves: V, the last price, per side the filled
// orders (the first of the list), and the orders filled or partly filled.
struct Match {
    int32_t V, last, full[2], touched;
};

// The matching of a step whose crossing orders go past the first 64 of a
// side, by one wave.
__device__ __noinline__ Match match_long(const uint64_t* list, const int32_t* o_price,
                                         int32_t* o_qty, int32_t* cum, uint32_t* abits, int32_t C,
                                         int32_t nb, int32_t ns, int32_t last) {
    const int lane = threadIdx.x & 63;
    // cumulative shares along the orders priced through the other side's best
    const int32_t best_bid = o_price[slot_of(list[0])];
    const int32_t best_ask = o_price[slot_of(list[C - 1])];
    int32_t cross[2];
    for (int s = 0; s < 2; ++s) {
        const int32_t n = s ? ns : nb, kbase = s ? C - 1 : 0, cbase = s ? C + 1 : 0;
        int32_t sum = 0, nx = 0;
        for (int32_t i0 = 0; i0 < n; i0 += 64) {
            const int32_t i = i0 + lane;
            int32_t q = 0;
            bool in = false;
            if (i < n) {
                const int32_t slot = slot_of(list[kbase + signed_pos(i, -s)]);
                const int32_t p = o_price[slot];
                in = s ? p <= best_bid : p >= best_ask;
                q = in ? o_qty[slot] : 0;
            }
            const int32_t incl = wave_incl_sum(q);
            if (in) cum[cbase + signed_pos(i, -s)] = sum + incl;
            const int32_t got = int32_t(__popcll(__ballot(in)));
            sum += __builtin_amdgcn_readlane(incl, 63);
            nx += got;
            if (got < 64) break;
        }
        cross[s] = nx;
    }
    wave_lds_sync();
    // V = max over the crossing buys of min(CB, CS(price))
    int32_t v = 0;
    for (int32_t i = lane; i < cross[0]; i += 64) {
        const int32_t pb = o_price[slot_of(list[i])];
        int32_t lo = 0, hi = cross[1];               // sells priced at most pb: [0, lo)
        while (lo < hi) {
            const int32_t mid = (lo + hi) >> 1;
            if (o_price[slot_of(list[C - 1 - mid])] <= pb) lo = mid + 1; else hi = mid;
        }
        const int32_t cs = lo > 0 ? cum[C + 1 - (lo - 1)] : 0;
        v = max(v, min(cum[i], cs));
    }
    Match r = {wave_max_nonneg(v), last, {0, 0}, 0};
    int32_t share[2] = {0, 0};
    for (int s = 0; s < 2; ++s) {
        const int32_t kbase = s ? C - 1 : 0, cbase = s ? C + 1 : 0;
        for (int32_t i0 = 0; i0 < cross[s] && r.V > 0; i0 += 64) {
            const int32_t i = i0 + lane;
            bool part = false, whole = false, covers = false;
            int32_t price = 0;
            if (i < cross[s]) {
                const int32_t slot = slot_of(list[kbase + signed_pos(i, -s)]);
                const int32_t q = o_qty[slot], incl = cum[cbase + signed_pos(i, -s)];
                const int32_t room = r.V - (incl - q);
                price = o_price[slot];
                if (room > 0) {
                    whole = room >= q;
                    part = !whole;
                    covers = r.V <= incl;
                    if (whole)
                        atomicAnd(&abits[slot >> 5], ~(1u << (slot & 31)));
                    else
                        o_qty[slot] = q - room;
                }
            }
            const uint64_t at = __ballot(covers);
            if (at) share[s] = __builtin_amdgcn_readlane(price, __ffsll((unsigned long long)at) - 1);
            const int32_t w = int32_t(__popcll(__ballot(whole)));
            r.full[s] += w;
            r.touched += w + int32_t(__popcll(__ballot(part)));
            if (w < 64) break;
        }
    }
    if (r.V > 0) r.last = int32_t((int64_t(share[0]) + share[1]) / 2);
    return r;
}

// The matching of a step, by one wave.  Along the buys CB grows and CS(price)
// falls, so V is reached at the first buy r with CB_r >= CS(p_r); it and the
// sells it needs are nearly always among the first 64 of each side (lane i:
// entry i).
__device__ __forceinline__ Match match_books(const uint64_t* list, const int32_t* o_price,
                                             int32_t* o_qty, int32_t* cum, uint32_t* abits,
                                             int32_t C, int32_t nb, int32_t ns, int32_t last) {
    const int lane = threadIdx.x & 63;
    int32_t pr[2], qt[2], inc[2], sl[2] = {0, 0};
    if (lane < nb) sl[0] = slot_of(list[lane]);
    if (lane < ns) sl[1] = slot_of(list[C - 1 - lane]);
#pragma unroll
    for (int w = 0; w < 2; ++w) {
        pr[w] = o_price[sl[w]];
        qt[w] = lane < (w ? ns : nb) ? o_qty[sl[w]] : 0;
    }
#pragma unroll
    for (int w = 0; w < 2; ++w) inc[w] = wave_incl_sum(qt[w]);
    // sells priced at most this lane's buy: c of the first 64 (their prices
    // ascend), cs shares
    int32_t c = 0;
    const int32_t sells = ns < 64 ? ns : 64;
#pragma unroll
    for (int h = 32; h >= 1; h >>= 1) {
        const int32_t p = __shfl(pr[1], c + h - 1, 64);
        c += c + h <= sells && p <= pr[0] ? h : 0;
    }
    c += c == 63 && sells == 64 && __builtin_amdgcn_readlane(pr[1], 63) <= pr[0] ? 1 : 0;
    const int32_t cs_at = __shfl(inc[1], c > 0 ? c - 1 : 0, 64);
    const int32_t cs = c > 0 ? cs_at : 0;
    const uint64_t met = __ballot(lane < nb && inc[0] >= cs);
    Match r = {0, last, {0, 0}, 0};
    bool more = false;                        // the first 64 do not settle it
    if (met) {
        const int at = __ffsll((unsigned long long)met) - 1;
        r.V = __builtin_amdgcn_readlane(cs, at);
        if (at > 0) r.V = max(r.V, __builtin_amdgcn_readlane(inc[0], at - 1));
        more = __builtin_amdgcn_readlane(c, at) == 64 && ns > 64;
    } else if (nb > 0) {
        // every CB below its CS (nb > 64: the list goes on)
        r.V = __builtin_amdgcn_readlane(inc[0], nb < 64 ? nb - 1 : 63);
        more = nb > 64;
    }
    if (more) return match_long(list, o_price, o_qty, cum, abits, C, nb, ns, last);
    if (r.V > 0) {
        // an order fills the part of its share range below V
        int32_t share[2];
#pragma unroll
        for (int w = 0; w < 2; ++w) {
            const int32_t room = r.V - (inc[w] - qt[w]);   // shares of V left for this order
            const bool in = lane < (w ? ns : nb) && room > 0;
            const bool whole = in && room >= qt[w];
            r.touched += int32_t(__popcll(__ballot(in)));
            r.full[w] = int32_t(__popcll(__ballot(whole)));
            // the order covering share V
            const uint64_t at = __ballot(in && r.V <= inc[w]);
            share[w] = at ? __builtin_amdgcn_readlane(pr[w], __ffsll((unsigned long long)at) - 1) : 0;
            if (whole) atomicAnd(&abits[sl[w] >> 5], ~(1u << (sl[w] & 31)));
            if (in && !whole) o_qty[sl[w]] = qt[w] - room;
        }
        r.last = int32_t((int64_t(share[0]) + share[1]) / 2);
    }
    return r;
}

// A trader's draws of one step: shares (21 bits from bit 0), price offset
// above last - spread (24 bits from bit 24).
__device__ __forceinline__ uint64_t trader_word(const LobArgs& a, uint64_t skey, int32_t tr,
                                                bool* want, bool* sell) {
    const uint32_t k = uint32_t(tr);
    *want = tr < a.traders && draw(skey, k, kLobOrder) < a.T_order;
    *sell = draw(skey, k, kLobSide) >= 0x80000000u;
    const uint32_t off = scale(draw(skey, k, kLobPrice), uint32_t(2 * a.spread + 1));
    const uint32_t qty = 1u + scale(draw(skey, k, kLobQty), uint32_t(a.max_qty));
    return uint64_t(qty) | (uint64_t(off) << 24);
}

// Ranks of this thread's first N keys among the m keys `all`.
constexpr int kPlaceTurns = kMaxCap / 64 / kSideWaves;

template <int N>
__device__ __forceinline__ void rank_keys(const uint64_t* all, int32_t m,
                                          const uint64_t (&key)[kPlaceTurns],
                                          int32_t (&rank)[kPlaceTurns]) {
#pragma unroll 4
    for (int32_t u = 0; u < m; ++u) {
        const uint64_t x = all[u];
#pragma unroll
        for (int p = 0; p < N; ++p) rank[p] += x < key[p] ? 1 : 0;
    }
}

// Puts the m new orders of a side (more than a wave has lanes for, or in a book
// with odd times) into its next list, by its four waves: their ranks among
// themselves, and the staying entries before each by the prefix sums of the
// histogram, made in place by the last wave.  The whole workgroup calls it (m = 0
// for a side that is done).  50 books of 1024 slots with 1024 traders x 1 step 52
// us, 93 with the last wave alone; 60 steps 0.80 ms, 1.09 so.
__device__ __noinline__ void place_many(const uint64_t* nkey, int32_t* hist, uint64_t* nxt,
                                        uint32_t* abits, int32_t m, int32_t nbase, int32_t hbase,
                                        int32_t kbase, int32_t neg, int w) {
    const int lane = threadIdx.x & 63;
    const int32_t dir = neg ? -1 : 1;
    uint64_t key[kPlaceTurns];
    int32_t rank[kPlaceTurns];
#pragma unroll
    for (int p = 0; p < kPlaceTurns; ++p) {
        const int32_t q = (p * kSideWaves + w) * 64 + lane;
        key[p] = q < m ? nkey[nbase + dir * q] : 0ull;
        rank[p] = 0;
    }
    const uint64_t* const all = nkey + (neg ? nbase - m + 1 : nbase);   // (in any order)
    if (m <= kSideWaves * 64)
        rank_keys<1>(all, m, key, rank);
    else if (m <= 2 * kSideWaves * 64)
        rank_keys<2>(all, m, key, rank);
    else
        rank_keys<kPlaceTurns>(all, m, key, rank);
    if (w == kSideWaves - 1) {
        int32_t carry = 0;
        for (int32_t r0 = 0; r0 < m; r0 += 64) {
            const int32_t r = r0 + lane;
            const int32_t in = wave_incl_sum(r < m ? hist[hbase + dir * r] : 0);
            if (r < m) hist[hbase + dir * r] = carry + in;
            carry += __builtin_amdgcn_readlane(in, 63);
        }
    }
    __syncthreads();
#pragma unroll
    for (int p = 0; p < kPlaceTurns; ++p) {
        if ((p * kSideWaves + w) * 64 + lane >= m) continue;
        const int32_t slot = slot_of(key[p]);
        atomicOr(&abits[slot >> 5], 1u << (slot & 31));
        nxt[kbase + signed_pos(rank[p] + hist[hbase + dir * rank[p]], neg)] = key[p];
    }
}

// One workgroup of eight waves owns a book for the whole call: waves 0-3 keep
// the buys' list, waves 4-7 the sells'.
//
// What bounds a step: the instructions on its longest chain of phases, not
// bytes (the book is in LDS; 64 bytes of statistics leave it a step).  A wave
// alone on its SIMD takes 6 to 10 cycles for an instruction here, while a
// barrier of eight waves takes about 35.  So the lists stay sorted from step
// to step and a step only merges its few dozen new orders in and matches the
// top of the book; each phase gives a wave one run of 64 list entries, with a
// barrier after it; and the draws, which depend on no state, are made for the
// next step by the waves that do not match.  500 books of 1000 slots with 100
// traders, 100 steps: 0.51 ms, where one workgroup of sixteen waves that ranked
// every order against its whole side in each step took 2.1 ms; four waves (two
// for the lists, two for the draws) take 0.58 ms.
__global__ __launch_bounds__(kBlock) void k_lob_run(LobArgs a) {
    extern __shared__ uint64_t lds64[];
    __shared__ uint64_t s_wm[2][kTraderChunks], s_sm[2][kTraderChunks];  // wants / sells, 64 traders
    __shared__ int32_t s_cnt[2][kListChunks + 1];   // survivors of each run of 64 entries
    __shared__ int32_t s_live[2], s_head[2];        // list lengths, filled entries at the front
    __shared__ int32_t s_new[2];                    // new orders per side
    __shared__ int32_t s_stat[kCols];
    __shared__ int32_t s_expired, s_load, s_odd;
    const int32_t C = a.cap, T = a.traders, M = new_max(C, T);
    uint64_t* const keys0 = lds64;
    uint64_t* const keys1 = keys0 + C;
    uint64_t* const nkey = keys1 + C;
    uint64_t* const words = nkey + M;         // [2][T]
    uint32_t* const nword0 = reinterpret_cast<uint32_t*>(
        (reinterpret_cast<uintptr_t>(words + 2 * T) + 15) & ~uintptr_t(15));
    int32_t* const o_price = reinterpret_cast<int32_t*>(nword0 + 2 * word_room(M));
    int32_t* const o_qty = o_price + C;
    int32_t* const o_time = o_qty + C;
    int32_t* const cum = o_time + C;          // C + 2
    int32_t* const hist = cum + C + 2;        // M + 2
    uint32_t* const abits = reinterpret_cast<uint32_t*>(hist + M + 2);
    uint16_t* const free_list = reinterpret_cast<uint16_t*>(abits + kBitWords);
    uint8_t* const placed_as = reinterpret_cast<uint8_t*>(free_list + M);   // in this call: 1 buy, 2 sell
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int s = wave / kSideWaves, w = wave % kSideWaves;           // side, wave within it
    const int32_t neg = -s, dir = s ? -1 : 1;
    const int32_t kbase = s ? C - 1 : 0;      // list position i of this side: kbase + dir * i
    const int32_t nbase = s ? M - 1 : 0;      // the same among the new orders
    const int32_t hbase = s ? M + 1 : 0;      // ... in the histogram
    const int32_t klane = kbase + dir * (w * 64 + lane);
    const int64_t base = int64_t(blockIdx.x) * C;
    const uint32_t seed = a.seed + blockIdx.x;
    int32_t last = a.last_price[blockIdx.x];
    // the traders' words and masks of one step, by `helpers` waves (this one is `h`)
    auto draw_orders = [&](int32_t step_k, int h, int helpers) {
        const uint64_t skey = stream_key(seed, a.step0 + uint32_t(step_k));
        const int buf = step_k & 1;
        for (int32_t c = h; c * 64 < T; c += helpers) {
            const int32_t tr = c * 64 + lane;
            bool want, sell;
            const uint64_t word = trader_word(a, skey, tr, &want, &sell);
            const uint64_t wm = __ballot(want), sm = __ballot(want && sell);
            if (want) words[buf * T + tr] = word;
            if (lane == 0) {
                s_wm[buf][c] = wm;
                s_sm[buf][c] = sm;
            }
        }
    };

    // ---- load the book; sort the live orders' keys (bitonic, in place in the
    // two list buffers, buys before sells by bit 63)
    for (int i = tid; i < kBitWords; i += kBlock) abits[i] = 0;
    if (tid == 0) {
        s_load = 0;
        s_odd = 0;
        s_expired = 0;
    }
    if (tid < 2) s_head[tid] = 0;
    if (tid < 2 * kTraderChunks) {
        s_wm[tid & 1][tid >> 1] = 0;
        s_sm[tid & 1][tid >> 1] = 0;
    }
    __syncthreads();
    draw_orders(0, wave, kWaves);
    for (int32_t i0 = 0; i0 < C; i0 += kBlock) {
        const int32_t i = i0 + tid;
        bool live = false, sell = false;
        if (i < C) {
            placed_as[i] = 0;
            o_price[i] = a.price[base + i];
            o_qty[i] = a.qty[base + i];
            o_time[i] = a.time[base + i];
            live = a.alive[base + i] != 0;
            sell = a.side[base + i] != 0;
        }
        const uint64_t lv = __ballot(live);
        int32_t at = 0;
        if (lane == 0) {
            at = atomicAdd(&s_load, int32_t(__popcll(lv)));
            if (i < C) abits[i >> 5] = uint32_t(lv);
            if (i + 32 < C) abits[(i >> 5) + 1] = uint32_t(lv >> 32);
        }
        at = __builtin_amdgcn_readfirstlane(at) + int32_t(lane_rank(lv));
        if (live) {
            keys0[at] = priority_key(sell, o_price[i], o_time[i], i);
            if (o_time[i] < 0 || o_time[i] >= int32_t(a.step0)) s_odd = 1;
        }
    }
    __syncthreads();
    const int32_t n0 = s_load;
    {
        int32_t P = 1;
        while (P < n0) P <<= 1;               // P < 2 n0 <= 2 C: both list buffers hold it
        for (int32_t i = n0 + tid; i < P; i += kBlock) keys0[i] = ~0ull;
        __syncthreads();
        for (int32_t k = 2; k <= P; k <<= 1)
            for (int32_t j = k >> 1; j > 0; j >>= 1) {
                for (int32_t q = tid; q < (P >> 1); q += kBlock) {
                    const int32_t lo = ((q & ~(j - 1)) << 1) | (q & (j - 1)), hi = lo | j;
                    const uint64_t x = keys0[lo], y = keys0[hi];
                    if ((x > y) == ((lo & k) == 0)) {
                        keys0[lo] = y;
                        keys0[hi] = x;
                    }
                }
                __syncthreads();
            }
        // buys are the keys without the side bit; the sells go to the buffer's end
        int32_t lo = 0, hi = n0;
        while (lo < hi) {
            const int32_t mid = (lo + hi) >> 1;
            if (keys0[mid] & kSellBit) hi = mid; else lo = mid + 1;
        }
        uint64_t mine[kMaxCap / kBlock];
#pragma unroll
        for (int c = 0; c < kMaxCap / kBlock; ++c) {
            const int32_t i = lo + c * kBlock + tid;
            mine[c] = i < n0 ? keys0[i] : 0ull;
        }
        __syncthreads();
#pragma unroll
        for (int c = 0; c < kMaxCap / kBlock; ++c) {
            const int32_t i = lo + c * kBlock + tid;
            if (i < n0) keys0[C - 1 - (i - lo)] = mine[c];
        }
        if (tid == 0) {
            s_live[0] = lo;
            s_live[1] = n0 - lo;
        }
        __syncthreads();
    }
    // (a caller's book may hold times that are not of an earlier step, which no
    // run of this library leaves: the shortcuts below that rest on it are off)
    const bool odd_times = __builtin_amdgcn_readfirstlane(s_odd) != 0;

    for (int32_t k = 0; k < a.n_steps; ++k) {
        const int32_t t = int32_t(a.step0 + uint32_t(k));
        uint64_t* const old = (k & 1) ? keys1 : keys0;
        uint64_t* const nxt = (k & 1) ? keys0 : keys1;
        const int32_t head = __builtin_amdgcn_readfirstlane(s_head[s]);
        const int32_t n = __builtin_amdgcn_readfirstlane(s_live[s]) - head;   // entries past it
        const int32_t kl = klane + dir * head;
        // the statistics of the step before
        if (k > 0 && a.stats && wave == kWaves - 1 && lane < kCols)
            a.stats[(int64_t(k - 1) * a.n_books + blockIdx.x) * kCols + lane] = s_stat[lane];
        // ---- expiry (t - time >= expiry): bit p of surv says that this
        // thread's entry of pass p (run p kSideWaves + w) stays
        uint32_t surv = 0;
        {
            const int32_t cutoff = t >= INT32_MIN + a.expiry ? t - a.expiry : INT32_MIN;
            for (int32_t p = 0; (p * kSideWaves + w) * 64 < n; ++p) {
                const int32_t i = (p * kSideWaves + w) * 64 + lane;
                bool on = i < n;
                if (on) {
                    const uint64_t key = old[kl + dir * p * kSideWaves * 64];
                    const int32_t slot = slot_of(key);
                    const int32_t tm = odd_times ? o_time[slot] : int32_t(key >> 15) & 0xFFFFFF;
                    on = odd_times ? int64_t(t) - tm < a.expiry : tm > cutoff;
                    if (!on) atomicAnd(&abits[slot >> 5], ~(1u << (slot & 31)));
                }
                surv |= on ? 1u << p : 0u;
                const int32_t kept = int32_t(__popcll(__ballot(on)));
                if (lane == 0) {
                    s_cnt[s][p * kSideWaves + w] = kept;
                    const int32_t in = n - (p * kSideWaves + w) * 64;
                    if (kept < min(in, 64)) atomicAdd(&s_expired, min(in, 64) - kept);
                }
            }
        }
        for (int32_t i = tid; i < M + 2; i += kBlock) hist[i] = 0;
        __syncthreads();
        // ---- free slots, in slot order: wave v lists those of rows v, v + 8
        int32_t n_free;
        {
            uint64_t f_word = 0;                           // lanes 0-15: free slots of row `lane`
            if (lane < kRows) {
                const int32_t left = C - lane * 64;
                const uint64_t in = left <= 0 ? 0ull : (left >= 64 ? ~0ull : (1ull << left) - 1);
                f_word = ~((uint64_t(abits[2 * lane + 1]) << 32) | abits[2 * lane]) & in;
            }
            const int32_t f = int32_t(__popcll(f_word));
            const int32_t incl = wave_incl_sum(f);
            n_free = __builtin_amdgcn_readlane(incl, 63);
            for (int r = wave; r * 64 < C; r += kWaves) {
                const int32_t before = r ? __builtin_amdgcn_readlane(incl, r - 1) : 0;
                if (before >= M) break;
                const uint32_t lo = uint32_t(__builtin_amdgcn_readlane(int32_t(uint32_t(f_word)), r));
                const uint32_t hi = uint32_t(__builtin_amdgcn_readlane(int32_t(uint32_t(f_word >> 32)), r));
                const uint64_t fw = (uint64_t(hi) << 32) | lo;
                const int32_t j = before + int32_t(lane_rank(fw));
                if (((fw >> lane) & 1) && j < M) free_list[j] = uint16_t(r * 64 + lane);
            }
        }
        __syncthreads();
        // ---- new orders: the trader of rank j among this step's orders (in
        // trader order) takes the j-th lowest free slot; waves 0 and 1 take
        // the traders in turns of 64
        int32_t n_new = 0;
        if (wave < 2) {
            int32_t at_b = 0, at_s = 0;                    // new orders of each side so far
            for (int32_t c0 = 0; c0 * 64 < T; c0 += 2) {
                // placed orders of both waves' traders: those of rank below n_free
                uint64_t placed[2], sells[2];
                int32_t first[2];
#pragma unroll
                for (int v = 0; v < 2; ++v) {
                    const uint64_t wm = s_wm[k & 1][c0 + v];
                    first[v] = n_new;
                    const int32_t j = n_new + int32_t(lane_rank(wm));
                    placed[v] = __ballot(((wm >> lane) & 1) && j < n_free);
                    sells[v] = placed[v] & s_sm[k & 1][c0 + v];
                    n_new += int32_t(__popcll(wm));
                }
                const uint64_t pm = wave ? placed[1] : placed[0], sm = wave ? sells[1] : sells[0];
                const int32_t b0 = int32_t(__popcll(placed[0] & ~sells[0]));
                const int32_t s0 = int32_t(__popcll(sells[0]));
                const int32_t j = (wave ? first[1] : first[0]) + int32_t(lane_rank(pm));
                if ((pm >> lane) & 1) {
                    const uint64_t word = words[(k & 1) * T + (c0 + wave) * 64 + lane];
                    const int32_t slot = free_list[j];
                    const int64_t p = int64_t(last) - a.spread + int64_t((word >> 24) & 0xFFFFFFu);
                    const int32_t price = int32_t(p < 1 ? 1 : (p > kMaxPrice ? kMaxPrice : p));
                    const bool sell = (sm >> lane) & 1;
                    o_price[slot] = price;
                    o_qty[slot] = int32_t(word & 0xFFFFFFu);
                    o_time[slot] = t;
                    placed_as[slot] = sell ? 2 : 1;
                    // new keys of a side in trader order
                    const int32_t q = sell ? at_s + (wave ? s0 : 0) + int32_t(lane_rank(sm))
                                     : at_b + (wave ? b0 : 0) + int32_t(lane_rank(pm & ~sm));
                    const uint64_t key = priority_key(sell, price, t, slot);
                    nkey[sell ? M - 1 - q : q] = key;
                    if (q < kWordRanks)
                        nword0[(sell ? word_room(M) : 0) + q] = price_of(key) << 8 | uint32_t(q);
                }
                at_b += b0 + int32_t(__popcll(placed[1] & ~sells[1]));
                at_s += s0 + int32_t(__popcll(sells[1]));
            }
            if (tid == 0) {
                s_new[0] = at_b;
                s_new[1] = at_s;
            }
            // pad the words to a group of eight with the largest
            const int32_t mine = wave ? at_s : at_b;
            if (mine + lane < ((mine + 7) & ~7) && mine + lane < word_room(M))
                nword0[(wave ? word_room(M) : 0) + mine + lane] = ~0u;
        }
        __syncthreads();
        // ---- merge.  An order that stays moves to the number of those staying
        // before it plus the number of new orders below it (`under`); the new
        // order of rank r goes after the r new ones below it and the staying
        // ones with at most r new orders below them (a histogram of `under`).
        // Every older order is below a new one of its price
        const int32_t m = __builtin_amdgcn_readfirstlane(s_new[s]);
        const int32_t runs = (n + 63) >> 6;
        const uint4* const nword = reinterpret_cast<const uint4*>(nword0 + s * word_room(M));
        // new orders' words below x (eight at a time; the padding is never below)
        auto words_below = [&](uint32_t x) {
            int32_t c = 0;
            for (int32_t u = 0; u < m; u += 8) {
                const uint4 v = nword[u >> 2], z = nword[(u >> 2) + 1];
                c += (v.x < x) + (v.y < x) + (v.z < x) + (v.w < x) + (z.x < x) + (z.y < x) +
                     (z.z < x) + (z.w < x);
            }
            return c;
        };
        const bool by_word = m <= kWordRanks && !odd_times;
        int32_t under[kMaxCap / 64 / kSideWaves];
#pragma unroll
        for (int p = 0; p < kMaxCap / 64 / kSideWaves; ++p) {
            under[p] = 0;
            if (p * kSideWaves + w >= runs) continue;
            const bool on = (surv >> p) & 1u;
            const uint64_t key = on ? old[kl + dir * p * kSideWaves * 64] : 0ull;
            if (by_word)
                under[p] = words_below(price_of(key) << 8);
            else
                for (int32_t u = 0; u < m; ++u) under[p] += nkey[nbase + dir * u] < key ? 1 : 0;
            if (on) atomicAdd(&hist[hbase + signed_pos(under[p], neg)], 1);
        }
        // the rank of each of up to 64 new orders, by the side's last wave
        uint64_t key0 = 0;
        int32_t rank0 = 0;
        const bool few = by_word && m <= 64;
        if (w == kSideWaves - 1 && few) {
            if (lane < m) {
                key0 = nkey[nbase + dir * lane];
                const int32_t slot = slot_of(key0);
                atomicOr(&abits[slot >> 5], 1u << (slot & 31));
            }
            rank0 = words_below(lane < m ? price_of(key0) << 8 | uint32_t(lane) : 0u);
        }
        __syncthreads();
        {
            // the runs' survivors before each run (lane c: run c)
            const int32_t kept = lane < runs ? s_cnt[s][lane] : 0;
            const int32_t incl = wave_incl_sum(kept);
            const int32_t stay = __builtin_amdgcn_readlane(incl, 63);
#pragma unroll
            for (int p = 0; p < kMaxCap / 64 / kSideWaves; ++p) {
                const int32_t c = p * kSideWaves + w;
                if (c >= runs) continue;
                const bool on = (surv >> p) & 1u;
                const int32_t before = c ? __builtin_amdgcn_readlane(incl, c - 1) : 0;
                const int32_t at = before + int32_t(lane_rank(__ballot(on))) + under[p];
                if (on) nxt[kbase + signed_pos(at, neg)] = old[kl + dir * p * kSideWaves * 64];
            }
            if (w == kSideWaves - 1) {
                if (few) {
                    const int32_t h = lane < m ? hist[hbase + dir * lane] : 0;
                    const int32_t upto = wave_incl_sum(h);        // lane r: the entries before rank r
                    const int32_t at = rank0 + __shfl(upto, rank0, 64);
                    if (lane < m) nxt[kbase + signed_pos(at, neg)] = key0;
                }
                if (lane == 0) s_live[s] = stay + m;
            }
        }
        __syncthreads();
        if (odd_times || s_new[0] > 64 || s_new[1] > 64) {
            place_many(nkey, hist, nxt, abits, few ? 0 : m, nbase, hbase, kbase, neg, w);
            __syncthreads();
        }
        // ---- matching by wave 0, the next step's draws by the others
        if (wave == 0) {
            __builtin_amdgcn_s_setprio(3);   // the step waits for this wave
            const int32_t nb = __builtin_amdgcn_readfirstlane(s_live[0]);
            const int32_t ns = __builtin_amdgcn_readfirstlane(s_live[1]);
            const Match r = match_books(nxt, o_price, o_qty, cum, abits, C, nb, ns, last);
            last = r.last;
            const int32_t placed = n_new < n_free ? n_new : n_free;
            if (lane == 0) {
                s_head[0] = r.full[0];
                s_head[1] = r.full[1];
                s_stat[kBuys] = nb - r.full[0];
                s_stat[kSells] = ns - r.full[1];
                s_stat[kPlaced] = placed;
                s_stat[kDropped] = n_new - placed;
                s_stat[kExpired] = s_expired;
                s_stat[kVolume] = r.V;
                s_stat[kFilled] = r.touched;
                s_stat[kPrice] = last;
                s_expired = 0;
            }
            __builtin_amdgcn_s_setprio(0);
        } else if (k + 1 < a.n_steps) {
            draw_orders(k + 1, wave - 1, kWaves - 1);
        }
        __syncthreads();
        last = __builtin_amdgcn_readfirstlane(s_stat[kPrice]);
    }
    if (a.n_steps > 0 && a.stats && tid < kCols)
        a.stats[(int64_t(a.n_steps - 1) * a.n_books + blockIdx.x) * kCols + tid] = s_stat[tid];
    // ---- write the book back: a slot placed in this call takes its new side,
    // price and time; the shares and the dead slots' alive = 0 may have changed
    for (int32_t i = tid; i < C; i += kBlock) {
        const bool live = (abits[i >> 5] >> (i & 31)) & 1u;
        a.qty[base + i] = o_qty[i];
        if (placed_as[i]) {
            a.side[base + i] = placed_as[i] - 1;
            a.price[base + i] = o_price[i];
            a.time[base + i] = o_time[i];
            a.alive[base + i] = live ? 1 : 0;
        } else if (!live) {
            a.alive[base + i] = 0;
        }
    }
    if (tid == 0) a.last_price[blockIdx.x] = last;
}

__global__ __launch_bounds__(256) void k_lob_clear(LobArgs a, int64_t n) {
    for (int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x; i < n; i += int64_t(gridDim.x) * 256) {
        a.side[i] = 0;
        a.price[i] = 0;
        a.qty[i] = 0;
        a.time[i] = 0;
        a.alive[i] = 0;
        if (i < a.n_books) a.last_price[i] = a.price0;
    }
}

int check_lob(const abm_lob_params* p, const abm_lob_state* s) {
    if (!p || !s) return fail(ABM_E_INVALID, "params or state is NULL");
    if (p->cap < 1 || p->cap > kMaxCap) return fail(ABM_E_INVALID, "cap must be in [1, 1024]");
    if (p->traders < 0 || p->traders > kMaxTraders)
        return fail(ABM_E_INVALID, "traders must be in [0, 1024]");
    if (p->spread < 0 || p->spread > (1 << 22)) return fail(ABM_E_INVALID, "spread must be in [0, 2^22]");
    if (p->max_qty < 1 || p->max_qty > (1 << 20)) return fail(ABM_E_INVALID, "max_qty must be in [1, 2^20]");
    if (p->expiry < 1) return fail(ABM_E_INVALID, "expiry must be >= 1");
    if (p->price0 < 1 || p->price0 > kMaxPrice) return fail(ABM_E_INVALID, "price0 must be in [1, 2^24)");
    if (s->n_books < 1 || s->n_books > (1 << 20)) return fail(ABM_E_INVALID, "n_books must be in [1, 2^20]");
    if (!s->side || !s->price || !s->qty || !s->time || !s->alive || !s->last_price)
        return fail(ABM_E_INVALID, "book array is NULL");
    return ABM_OK;
}

LobArgs lob_args(const abm_lob_params* p, const abm_lob_state* s) {
    LobArgs a;
    a.cap = p->cap;
    a.traders = p->traders;
    a.T_order = p->T_order;
    a.spread = p->spread;
    a.max_qty = p->max_qty;
    a.expiry = p->expiry;
    a.price0 = p->price0;
    a.seed = p->seed;
    a.side = s->side;
    a.price = s->price;
    a.qty = s->qty;
    a.time = s->time;
    a.alive = s->alive;
    a.last_price = s->last_price;
    a.stats = s->stats;
    a.n_books = s->n_books;
    a.step0 = s->step;
    a.n_steps = 0;
    return a;
}

}  // namespace
}  // namespace abm

using namespace abm;

extern "C" int abm_lob_init(const abm_lob_params* p, abm_lob_state* s, void* stream) {
    int rc = check_lob(p, s);
    if (rc != ABM_OK) return rc;
    rc = check_device();
    if (rc != ABM_OK) return rc;
    LobArgs a = lob_args(p, s);
    const int64_t n = int64_t(s->n_books) * p->cap;
    const int64_t m = n > s->n_books ? n : s->n_books;
    const int64_t blocks = (m + 255) / 256 < 4096 ? (m + 255) / 256 : 4096;
    hipLaunchKernelGGL(k_lob_clear, dim3(uint32_t(blocks)), dim3(256), 0, as_stream(stream), a, m);
    rc = launch_status("lob_init");
    if (rc == ABM_OK) s->step = 0;
    return rc;
}

extern "C" int abm_lob_step(const abm_lob_params* p, abm_lob_state* s, int32_t n_steps,
                            void* stream) {
    int rc = check_lob(p, s);
    if (rc != ABM_OK) return rc;
    if (n_steps < 0) return fail(ABM_E_INVALID, "n_steps must be >= 0");
    if (uint64_t(s->step) + uint64_t(n_steps) > (1u << 24))
        return fail(ABM_E_INVALID, "steps beyond 2^24 are not supported (order times are 24-bit keys)");
    rc = check_device();
    if (rc != ABM_OK) return rc;
    if (n_steps == 0) return ABM_OK;
    LobArgs a = lob_args(p, s);
    a.n_steps = n_steps;
    hipLaunchKernelGGL(k_lob_run, dim3(uint32_t(s->n_books)), dim3(kBlock),
                       lob_lds_bytes(p->cap, p->traders), as_stream(stream), a);
    rc = launch_status("lob_step");
    if (rc == ABM_OK) s->step += uint32_t(n_steps);
    return rc;
}
