// batched.hip -- many independent predation models of uneven sizes in one
// persistent launch (the MI355X counterpart of vectorising whole models,
// paper Sec. 2 and Table 2, without requiring equal shapes).
//
// Each model is advanced by ONE workgroup for all of its steps, so every
// phase boundary is a workgroup barrier instead of a kernel launch; models too
// large for that are advanced side by side by launches over the whole device
// (launch_wide) or, in runs of very many steps, by teams of workgroups.  Workgroups
// take models from a queue in a host-chosen order (largest first) until the
// queue is empty; a model whose work is done is skipped.
//
// Per step, three passes over the model's slots in chunks of blockDim x ITEMS
// (below each range's high-water mark, see model_step):
//   A  move + claims   live agents move, pay one energy and post packed
//                      (tag, draw, slot) keys by 64-bit atomicMin into the
//                      three claim words of their cell (grass, prey, eater);
//   B  eat + breeders  each live agent compares its keys with the reduced
//                      words; grass winners gain and set the cell's regrowth
//                      step, eaten sheep are marked alive = 2 (dead, claims not
//                      yet cleared); breeders are compacted in slot order;
//                      (multi-prey models: in A the agents push themselves onto
//                      lists of their cell instead of posting prey and eater
//                      keys, and a pass between A and B pairs each cell's
//                      wolves and sheep by rank; see prey_match)
//   C  breed           free slots (alive 0 or 2) are ranked, the free slot of
//                      rank j < #breeders pulls its child from breeder j, and
//                      live agents with negative energy die.
// Claim keys carry a step tag (see tagged_key): within a period of steps a
// word left by an earlier step reads as unclaimed and loses to every fresh
// key, so the model's claim table is re-armed (streamed back to all-ones) only
// in pass C of a period's last step and of the last step a launch runs, which
// keeps the tables all-ones between launches.
// A model run by one workgroup whose claim table (three words per cell) fits
// in the workgroup's dynamic LDS keeps it there (LOCAL): the table is set to
// all-ones when the model is taken, pass A posts into it with LDS atomics, and
// pass C clears it whole every step.  The global table of such a model is not touched.  The launch
// gives each workgroup the LDS its occupancy leaves free, so no workgroup
// is displaced for it.
// Models of up to 256 x 256 cells whose live agents fit are taken before that
// by workgroups that hold the whole model in LDS (k_batched_chip, see
// onchip.hpp); what does not fit, or outgrows it, is left to the passes above.
// Grass is stored as the step at which a cell is grown again (0 = grown from
// the start), so the per-cell regrowth pass of the one-model path disappears:
// a cell is grown at step t iff ready <= t; eating at step t sets ready = t + R.
// The countdown of the model definition is max(0, ready - steps_done).
#include <hip/hip_runtime.h>

#include <atomic>

#include "abm.h"
#include "common.hpp"
#include "rng.hpp"
#include "scan.hpp"

namespace abm {
namespace {

constexpr uint64_t kNoClaim = ~0ull;
constexpr uint32_t kTagBits = 4;     // claim-key tag: periods of 14 steps
constexpr uint32_t kDxPacked = 0x9224u;  // see predation.hip: dir -> dx + 1, 2 bits each
constexpr uint32_t kDyPacked = 0xA940u;

// Words of the workspace header: the queues of the team models, of the models
// of one workgroup and of those run on the chip (by size class), the lengths of
// the lists k_classify makes of the latter two, the number of wide models and the
// most steps that one of them has.
constexpr int kChipClasses = 3;
enum QueueWord : int {
    kQueueTeam = 0, kQueueSolo, kSoloModels, kQueueChip, kChipModels = kQueueChip + kChipClasses,
    kWideModels = kChipModels + kChipClasses, kWideMostSteps, kQueueWords
};

// Cells plus slots from which a model of one workgroup that does not fit the
// chip joins the large ones (see launch_wide): one workgroup takes some 0.06 ms
// a step for it and more as it grows, which the launches' total no longer hides.
constexpr int64_t kWideSize = 1 << 15;
// Leading models of the order that may join them beside the teams' (200 models of
// 300^2 to 430^2 cells, 15 of them a team's, x 20 steps: 11.3 ms with 64, the others
// one workgroup each afterwards, 10.0 with all of them).
constexpr int32_t kWideAtLeast = 256;
// Steps of a run up to which it is done by launches: three or four are queued
// for each of the max_steps steps, whether or not the models have that many
// left (about 2.5 us a launch that finds nothing to do).  A recorded run keeps
// them as graph nodes.
constexpr int32_t kWideSteps = 256, kWideStepsRecorded = 64;

struct BatchArgs {
    abm_model_desc* models;
    const int32_t* order;      // queue order of model indices
    int32_t n_models;
    int32_t max_steps;         // per model, this launch
    int32_t* ready;            // packed per-cell regrowth step
    uint64_t* claims;          // packed, 3 words per cell
    int32_t *sx, *sy, *se, *sa;
    int32_t *wx, *wy, *we, *wa;
    uint32_t* queue;           // model queue counters (see QueueWord; reset before the launch)
    int32_t listed;            // the models of one workgroup come from the lists of k_classify
    int32_t chip_bytes[kChipClasses];   // LDS of a workgroup of k_batched_chip (0: class not used)
    int64_t* chip_list[kChipClasses];   // models | steps << 32 (the last class: in the descriptors)
    uint8_t* wide;             // order[n_team, n_wide): taken by launch_wide (written by k_classify)
    int32_t n_wide;            // 0: none
    int32_t* scratch;          // per-workgroup breeder list
    int64_t scratch_stride;    // ints per workgroup
    uint64_t* err;             // workspace error word
    int32_t *link_s, *link_w;  // per-cell list links of multi-prey models (or null)
    int32_t n_team;            // order[0, n_team) run in teams
    int32_t lds_words;         // dynamic LDS claim words per workgroup (0: none)
    uint32_t team_k;           // members per team
    uint32_t team_wgs;         // workgroups in teams (multiple of 8 * team_k)
    uint32_t* team_ctr;        // barrier counter per team
    int32_t* team_mail;        // model mailbox per team
    int32_t* team_counts;      // [workgroup][5] member counts
};

__device__ __forceinline__ int32_t wrap_step(int32_t v, int32_t d, int32_t n) {
    v += d;
    return v < 0 ? n - 1 : (v >= n ? 0 : v);
}

__device__ __forceinline__ uint64_t ld_claim(const uint64_t* p) {
    // atomics execute in L2; a plain load could hit a stale line in the CU's L1
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void claim_min(uint64_t* p, uint64_t key) {
    atomicMin(reinterpret_cast<unsigned long long*>(p), static_cast<unsigned long long>(key));
}

// A claim posted into the LOCAL table, through an LDS-qualified pointer (a
// generic pointer into LDS does not compile for this atomic here).
__device__ __forceinline__ void claim_min_lds(uint64_t* p, uint64_t key) {
    typedef __attribute__((address_space(3))) unsigned long long lds_u64;
    __hip_atomic_fetch_min((lds_u64*)p, static_cast<unsigned long long>(key), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Makes `word` (a slot with the step's tag) the head of the list whose head
// is *p; returns the previous head.
__device__ __forceinline__ uint64_t push_head(uint64_t* p, uint64_t word) {
    return __hip_atomic_exchange(p, word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ uint64_t push_head_lds(uint64_t* p, uint64_t word) {
    typedef __attribute__((address_space(3))) unsigned long long lds_u64;
    return __hip_atomic_exchange((lds_u64*)p, static_cast<unsigned long long>(word),
                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

__device__ __forceinline__ void rearm(uint64_t* p) {
    __hip_atomic_store(p, kNoClaim, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The LOCAL claim table: the workgroup's dynamic LDS.
__device__ __forceinline__ uint64_t* local_claims() {
    extern __shared__ uint64_t dyn_claims[];
    return dyn_claims;
}

__device__ __forceinline__ void local_fill(uint64_t* lc, int32_t words) {
    for (int32_t i = threadIdx.x; i < words; i += blockDim.x) lc[i] = kNoClaim;
}

// (tag, draw, slot) from the high bits down: within a step these order as
// (draw, slot), the method's claim order; an earlier step of the period has
// a larger tag, so its words lose to fresh keys and read as unclaimed.
__device__ __forceinline__ uint64_t tagged_key(uint64_t tag_hi, uint32_t sb, uint64_t skey,
                                               int64_t slot, uint32_t purpose) {
    return tag_hi | (uint64_t(draw(skey, uint32_t(slot), purpose)) << sb) | uint64_t(slot);
}

// The ranking order of multi-prey (no tag: only keys of one step are compared).
__device__ __forceinline__ uint64_t key_of(uint64_t skey, int64_t slot, uint32_t purpose) {
    return (uint64_t(draw(skey, uint32_t(slot), purpose)) << 32) | uint32_t(slot);
}

__device__ __forceinline__ uint32_t block_sum32(uint32_t v, uint32_t* lds) {
    v = wave_sum(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = v;
    __syncthreads();
    uint32_t s = 0;
    for (int w = 0; w < int(blockDim.x >> 6); ++w) s += lds[w];
    return s;
}

// Block-wide maximum of one value per thread (every thread gets it); lds
// holds one word per wave.  Two barriers.
__device__ __forceinline__ int32_t block_max32(int32_t v, uint32_t* lds) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v = max(v, __shfl_xor(v, o, 64));
    __syncthreads();
    if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = uint32_t(v);
    __syncthreads();
    int32_t m = int32_t(lds[0]);
    for (int w = 1; w < int(blockDim.x >> 6); ++w) m = max(m, int32_t(lds[w]));
    return m;
}

// Block-wide inclusive scan of one value per thread: *incl gets this thread's
// inclusive prefix, the return value the block total.  lds holds one word per
// wave.
__device__ __forceinline__ uint32_t block_incl_scan32(uint32_t v, uint32_t* lds, uint32_t* incl) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    __syncthreads();
    if (lane == 63) lds[wave] = x;
    __syncthreads();
    uint32_t before = 0, all = 0;
    for (int w = 0; w < int(blockDim.x >> 6); ++w) {
        const uint32_t s = lds[w];
        before += w < wave ? s : 0u;
        all += s;
    }
    *incl = before + x;
    return all;
}

// Block-wide exclusive ranks of ITEMS flags per lane over one chunk (slot
// order = wave, item, lane); returns the chunk total.  lds holds one word per
// wave.  Two barriers.
template <int ITEMS>
__device__ __forceinline__ uint32_t chunk_rank(const bool (&f)[ITEMS], uint32_t (&rank)[ITEMS],
                                               uint32_t* lds) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t run = 0;
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        const uint64_t b = __ballot(f[k]);
        rank[k] = run + lane_rank(b);
        run += static_cast<uint32_t>(__popcll(b));
    }
    __syncthreads();
    if (lane == 0) lds[wave] = run;
    __syncthreads();
    uint32_t before = 0, all = 0;
    const int nw = blockDim.x >> 6;
    for (int w = 0; w < nw; ++w) {
        const uint32_t v = lds[w];
        before += w < wave ? v : 0u;
        all += v;
    }
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) rank[k] += before;
    return all;
}

struct ModelView {
    int32_t W, H, R, gain[2];
    uint32_t T[2], seed;
    bool multi;                  // prey matched by rank within a cell
    uint32_t sb;                 // slot bits of a claim key
    uint32_t period;             // steps per tag period
    uint64_t tag_top;            // the first tag of a period
    uint64_t tag_mask;           // the tag field and the bits above it
    int32_t cap[2];
    int32_t* link[2];            // list links (multi), per species
    int32_t* ready;              // per cell the step, less `base`, at which it is grown
    int32_t base;
    uint64_t* claims;
    int32_t *x[2], *y[2], *e[2], *al[2];
};

__device__ __forceinline__ bool on_grid(const ModelView& v, int32_t x, int32_t y) {
    return x >= 0 && x < v.W && y >= 0 && y < v.H;
}

}  // namespace
}  // namespace abm

#include "onchip.hpp"

namespace abm {
namespace {

// A team of K workgroups advancing one model together (K = 1: one workgroup
// alone).  Member r owns the r-th contiguous K-th of each species' slots and
// keeps its own breeder list; members exchange per-range counts.  Members of a
// team are the workgroups base, base + 8, ..., base + 8 (K - 1): workgroups are
// dispatched to the eight XCDs in turn, so the members normally share one L2.
// Correctness does not rest on that: the team barrier uses agent-scope fences.
constexpr int kMaxTeam = 16;
constexpr int kCountWords = 5;   // breeders of both species, free slots of both, live
constexpr int kMaxWorkgroups = 8 * 1024;

struct Team {
    int K, r;
    uint32_t gen;               // team barriers passed
    uint32_t* ctr;              // barrier counter (K > 1)
    int32_t* scratch;           // lists of all workgroups
    int64_t stride;             // ints per list
    int32_t* counts;            // [workgroup][kCountWords]
    uint32_t base;              // workgroup index of member 0
    uint64_t* err;
    int32_t* s_pre;             // LDS: breeder prefixes [2][kMaxTeam + 1], free prefix [2], live
    int32_t* s_ok;              // LDS: barrier outcome
    int32_t* s_bound;           // LDS: [2][kMaxTeam + 1] member range bounds of this launch
    int32_t* s_mark;            // LDS: [2] per species, 1 + the member's highest live slot after
                                // the last step (no live agent at or above it), or INT32_MAX
};

__device__ __forceinline__ int32_t* member_list(const Team& tm, int j) {
    return tm.scratch + int64_t(tm.base + 8u * uint32_t(j)) * tm.stride;
}

// Team-wide barrier; false if a member never arrived (the error word is set).
// Every wave waits until its own stores are performed at the L2, then the
// workgroup barrier; thread 0 alone makes the L2 contents visible device-wide
// (agent-scope release), counts the member in, waits for the others and
// acquires (agent scope, which also drops the CU's stale L1 lines) before the
// second workgroup barrier releases the other waves.  One release per member
// instead of one per wave: every wave writing back the L2 costs ~10x more
// when hundreds of workgroups are resident.
__device__ __forceinline__ bool team_sync(Team& tm) {
    if (tm.K == 1) {
        __syncthreads();
        return true;
    }
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (threadIdx.x == 0) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        __hip_atomic_fetch_add(tm.ctr, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const uint32_t target = (tm.gen + 1) * uint32_t(tm.K);
        int32_t ok = 1;
        uint32_t spins = 0;
        while (__hip_atomic_load(tm.ctr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target) {
            if (++spins > kSpinLimit) {
                st_agent(tm.err, 1ull);
                ok = 0;
                break;
            }
            __builtin_amdgcn_s_sleep(1);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        *tm.s_ok = ok;
    }
    __syncthreads();
    ++tm.gen;
    return *tm.s_ok != 0;
}

// Multi-prey rule for wolf j whose cell's words are cw (Sec. 4, Alg. 1 applied
// within one cell): j has rank r among the cell's wolves by eat key and takes
// the sheep of rank r among the cell's sheep by prey key, if there is one,
// marking it alive = 2 and gaining.  Ranks are counted by walking the cell's
// lists, whose heads are the prey (sheep) and eater (wolf) words; distinct
// wolves have distinct ranks, so no sheep is taken twice.  Quadratic in the
// sheep of one cell, which are few at the workloads' densities.
template <class Read, class Head>
__device__ __forceinline__ void prey_match(const ModelView& v, uint64_t skey, const uint64_t* cw,
                                           int32_t j, Read rd, Head head) {
    const int32_t first = head(rd(cw + 1));
    if (first < 0) return;
    const uint64_t mine = key_of(skey, j, kWolfEatKey);
    uint32_t r = 0;
    for (int32_t w = head(rd(cw + 2)); w >= 0; w = v.link[1][w])
        r += key_of(skey, w, kWolfEatKey) < mine ? 1u : 0u;
    for (int32_t q = first; q >= 0; q = v.link[0][q]) {
        const uint64_t kq = key_of(skey, q, kSheepPreyKey);
        uint32_t below = 0;
        for (int32_t u = first; u >= 0; u = v.link[0][u])
            below += key_of(skey, u, kSheepPreyKey) < kq ? 1u : 0u;
        if (below == r) {
            v.al[0][q] = 2;
            v.e[1][j] += v.gain[1];
            return;
        }
    }
}

// One step t of model v by team tm; false if the team barrier failed.  A chunk
// is blockDim * ITEMS slots; item k of lane l of wave w is slot
// c0 + (w * ITEMS + k) * 64 + l, so each load instruction of a wave covers 64
// consecutive slots and the ITEMS loads of a lane are issued together.
// A step's statistics of a model of one workgroup, added up in LDS.
struct StepCounts {
    int32_t live[2], grass, eaten, births[2], starved[2];
};

template <int ITEMS, bool LOCAL>
__device__ bool model_step(const ModelView& v, uint32_t t, uint32_t t0, bool last, Team& tm,
                           uint32_t* lds, uint32_t* live_out, StepCounts* counts = nullptr) {
    uint64_t* const claims = LOCAL ? local_claims() : v.claims;
    // LOCAL: the atomics of pass A are complete at the barrier that ends it
    auto rd = [](const uint64_t* p) { return LOCAL ? *p : ld_claim(p); };
    auto post = [](uint64_t* p, uint64_t key) {
        if constexpr (LOCAL)
            claim_min_lds(p, key);
        else
            claim_min(p, key);
    };
    // wave-uniform: kept in scalar registers
    const uint32_t phase = __builtin_amdgcn_readfirstlane((t - t0) % v.period);
    const uint32_t sb = __builtin_amdgcn_readfirstlane(v.sb);
    const uint64_t tag_hi =
        uint64_t(__builtin_amdgcn_readfirstlane(uint32_t(v.tag_top - phase) << sb)) << 32;
    const uint64_t tag_mask =
        uint64_t(__builtin_amdgcn_readfirstlane(uint32_t(v.tag_mask >> 32))) << 32;
    auto claimed = [tag_hi, tag_mask](uint64_t w) { return (w & tag_mask) == tag_hi; };
    // a list head's slot, or -1 (a word of an earlier step, or all-ones: the end)
    auto head = [tag_hi, tag_mask](uint64_t w) {
        return (w & tag_mask) == tag_hi ? int32_t(w & ~tag_mask) : -1;
    };
    // multi-prey: the agent's link is the cell's previous head
    auto push = [tag_hi, head](uint64_t* p, int32_t slot, int32_t* link) {
        const uint64_t word = tag_hi | uint64_t(uint32_t(slot));
        const uint64_t prev = LOCAL ? push_head_lds(p, word) : push_head(p, word);
        link[slot] = head(prev);
    };
    const uint64_t skey = stream_key(v.seed, t);
    const uint32_t move_p[2] = {kSheepMove, kWolfMove};
    const uint32_t breed_p[2] = {kSheepBreed, kWolfBreed};
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int32_t chunk = int32_t(blockDim.x) * ITEMS;
    const int32_t lbase = wave * ITEMS * 64 + lane;
    // this member's slot range of each species (the whole model when alone, the
    // launch's balanced bounds in a team); species 1's list follows species 0's
    int32_t lo[2], hi[2];
    if (tm.K == 1) {
        lo[0] = 0;
        hi[0] = v.cap[0];
        lo[1] = 0;
        hi[1] = v.cap[1];
    } else {
        lo[0] = tm.s_bound[tm.r];
        hi[0] = tm.s_bound[tm.r + 1];
        lo[1] = tm.s_bound[kMaxTeam + 1 + tm.r];
        hi[1] = tm.s_bound[kMaxTeam + 1 + tm.r + 1];
    }
    const int32_t list1 = v.cap[0];
    int32_t* my_list = member_list(tm, tm.r);
    // passes A and B visit [lo, eff): every live agent of the range lies below
    // the mark the last step left.  Each wave copies the mark into registers
    // here, after the barrier that ended the last step, and the mark is written
    // again only after every loop of this step (behind the barriers of the
    // reduction that computes it), so every wave runs the same trip counts.
    int32_t eff[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const int32_t mk = tm.s_mark[s];
        eff[s] = __builtin_amdgcn_readfirstlane(max(lo[s], min(hi[s], mk)));
    }

    // ---- A: move + claims
    uint32_t live = 0;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        for (int32_t c0 = lo[s]; c0 < eff[s]; c0 += chunk) {
            int32_t al[ITEMS];
#pragma unroll
            for (int k = 0; k < ITEMS; ++k) {
                const int32_t i = c0 + lbase + k * 64;
                al[k] = i < eff[s] ? v.al[s][i] : 0;
            }
#pragma unroll
            for (int k = 0; k < ITEMS; ++k) {
                if (al[k] == 0) continue;
                const int32_t i = c0 + lbase + k * 64;
                if (al[k] == 2) v.al[s][i] = 1;   // (the caller's: not the mark of pass B)
                ++live;
                if (counts) atomicAdd(&counts->live[s], 1);
                const uint32_t d = draw(skey, uint32_t(i), move_p[s]) >> 29;
                const int32_t x =
                    wrap_step(v.x[s][i], int32_t((kDxPacked >> (2 * d)) & 3u) - 1, v.W);
                const int32_t y =
                    wrap_step(v.y[s][i], int32_t((kDyPacked >> (2 * d)) & 3u) - 1, v.H);
                v.x[s][i] = x;
                v.y[s][i] = y;
                v.e[s][i] -= 1;
                if (!on_grid(v, x, y)) continue;
                const int64_t c = int64_t(y) * v.W + x;
                uint64_t* cw = claims + 3 * c;
                if (s == 0) {
                    if (v.ready[c] <= int32_t(t) - v.base)
                        post(cw + 0, tagged_key(tag_hi, sb, skey, i, kSheepGrassKey));
                    if (v.multi)
                        push(cw + 1, i, v.link[0]);
                    else
                        post(cw + 1, tagged_key(tag_hi, sb, skey, i, kSheepPreyKey));
                } else if (v.multi) {
                    push(cw + 2, i, v.link[1]);
                } else {
                    post(cw + 2, tagged_key(tag_hi, sb, skey, i, kWolfEatKey));
                }
            }
        }
    }
    live = block_sum32(live, lds);
    if (!team_sync(tm)) return false;    // every claim of the step is posted

    // ---- multi-prey: wolves of this member take their prey
    if (v.multi) {
        for (int32_t c0 = lo[1]; c0 < eff[1]; c0 += chunk) {
#pragma unroll
            for (int k = 0; k < ITEMS; ++k) {
                const int32_t j = c0 + lbase + k * 64;
                if (j >= eff[1] || v.al[1][j] == 0) continue;
                const int32_t x = v.x[1][j], y = v.y[1][j];
                if (!on_grid(v, x, y)) continue;
                prey_match(v, skey, claims + 3 * (int64_t(y) * v.W + x), j, rd, head);
            }
        }
        if (!team_sync(tm)) return false;   // eaten sheep and wolves' gains are visible
    }

    // ---- B: eat, member-local breeder lists (ascending), free-slot counts
    uint32_t nb_local[2], nf_local[2], nf_below[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        uint32_t base_rank = 0, nfree = 0;
        int32_t* list = my_list + (s ? list1 : 0);
        for (int32_t c0 = lo[s]; c0 < eff[s]; c0 += chunk) {
            int32_t al[ITEMS];
#pragma unroll
            for (int k = 0; k < ITEMS; ++k) {
                const int32_t i = c0 + lbase + k * 64;
                al[k] = i < eff[s] ? v.al[s][i] : 0;
            }
            bool br[ITEMS];
#pragma unroll
            for (int k = 0; k < ITEMS; ++k) {
                br[k] = false;
                const int32_t i = c0 + lbase + k * 64;
                if (al[k] == 0) {
                    nfree += i < eff[s] ? 1u : 0u;
                    continue;
                }
                const int32_t x = v.x[s][i], y = v.y[s][i];
                int32_t e = v.e[s][i];
                bool eaten = false;
                if (on_grid(v, x, y)) {
                    const int64_t c = int64_t(y) * v.W + x;
                    const uint64_t* cw = claims + 3 * c;
                    if (s == 0) {
                        if (rd(cw + 0) == tagged_key(tag_hi, sb, skey, i, kSheepGrassKey)) {
                            e += v.gain[0];
                            v.e[0][i] = e;
                            v.ready[c] = int32_t(t) - v.base + v.R;
                            if (counts) atomicAdd(&counts->grass, 1);
                        }
                        if (v.multi) {
                            eaten = al[k] == 2;   // taken by a wolf of its cell
                        } else if (claimed(rd(cw + 2)) &&
                                   rd(cw + 1) == tagged_key(tag_hi, sb, skey, i, kSheepPreyKey)) {
                            v.al[0][i] = 2;   // eaten: dead, its claims still to be reset
                            eaten = true;
                        }
                        nfree += eaten ? 1u : 0u;
                        if (counts && eaten) atomicAdd(&counts->eaten, 1);
                    } else if (!v.multi && claimed(rd(cw + 1)) &&
                               rd(cw + 2) == tagged_key(tag_hi, sb, skey, i, kWolfEatKey)) {
                        e += v.gain[1];
                        v.e[1][i] = e;
                    }
                }
                br[k] = !eaten && e > 0 && draw(skey, uint32_t(i), breed_p[s]) < v.T[s];
            }
            uint32_t rank[ITEMS];
            const uint32_t tot = chunk_rank<ITEMS>(br, rank, lds);
#pragma unroll
            for (int k = 0; k < ITEMS; ++k)
                if (br[k]) list[base_rank + rank[k]] = c0 + lbase + k * 64;
            base_rank += tot;
        }
        nb_local[s] = base_rank;
        nf_below[s] = block_sum32(nfree, lds);
        nf_local[s] = nf_below[s] + uint32_t(hi[s] - eff[s]);   // slots past the mark are free
    }
    // s_pre: [0, K] breeder prefix of species 0, [K+1, 2K+1] of species 1,
    // then the free-slot prefix of this member for both species and the live total
    int32_t* bpre0 = tm.s_pre;
    int32_t* bpre1 = tm.s_pre + tm.K + 1;
    int32_t* fpre = tm.s_pre + 2 * (tm.K + 1);
    if (tm.K == 1) {
        if (threadIdx.x == 0) {
            bpre0[0] = 0;
            bpre0[1] = int32_t(nb_local[0]);
            bpre1[0] = 0;
            bpre1[1] = int32_t(nb_local[1]);
            fpre[0] = 0;
            fpre[1] = 0;
            fpre[2] = int32_t(live);
        }
        __syncthreads();
    } else {
        if (threadIdx.x == 0) {
            int32_t* cnt = tm.counts + int64_t(tm.base + 8u * uint32_t(tm.r)) * kCountWords;
            cnt[0] = int32_t(nb_local[0]);
            cnt[1] = int32_t(nb_local[1]);
            cnt[2] = int32_t(nf_local[0]);
            cnt[3] = int32_t(nf_local[1]);
            cnt[4] = int32_t(live);
        }
        if (!team_sync(tm)) return false;   // every member's list and counts are visible
        if (threadIdx.x == 0) {
            int32_t b0 = 0, b1 = 0, f0 = 0, f1 = 0, lv = 0;
            for (int j = 0; j < tm.K; ++j) {
                const int32_t* cnt = tm.counts + int64_t(tm.base + 8u * uint32_t(j)) * kCountWords;
                bpre0[j] = b0;
                bpre1[j] = b1;
                b0 += cnt[0];
                b1 += cnt[1];
                if (j < tm.r) {
                    f0 += cnt[2];
                    f1 += cnt[3];
                }
                lv += cnt[4];
            }
            bpre0[tm.K] = b0;
            bpre1[tm.K] = b1;
            fpre[0] = f0;
            fpre[1] = f1;
            fpre[2] = lv;
        }
        __syncthreads();
    }
    *live_out = uint32_t(fpre[2]);

    int32_t top[2] = {0, 0};   // 1 + the highest slot this thread leaves alive
    // ---- C: breed into free slots, starve; re-arm the claims (every read of
    // the table in B is behind the barrier above): LOCAL every step, else at
    // the end of a tag period and at the last step of the launch, each team
    // member its share of the table
    if constexpr (LOCAL) {
        local_fill(claims, 3 * v.W * v.H);
    } else if (phase == v.period - 1 || last) {
        const int64_t words = 3 * int64_t(v.W) * v.H;
        const int64_t w0 = words * tm.r / tm.K, w1 = words * (tm.r + 1) / tm.K;
        for (int64_t w = w0 + threadIdx.x; w < w1; w += blockDim.x) rearm(claims + w);
    }
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const int32_t* bpre = s ? bpre1 : bpre0;
        const uint32_t nb = uint32_t(bpre[tm.K]);
        const int32_t list_off = s ? list1 : 0;
        uint32_t base_rank = uint32_t(fpre[s]);
        // births into this range: its free slots of model rank below nb; the
        // ones past the free slots below the mark take [eff, eff + above)
        const int64_t into = min(max(int64_t(nb) - int64_t(fpre[s]), int64_t(0)),
                                 int64_t(nf_local[s]));
        const int32_t above = int32_t(max(into - int64_t(nf_below[s]), int64_t(0)));
        const int32_t end = __builtin_amdgcn_readfirstlane(min(hi[s], eff[s] + above));
        for (int32_t c0 = lo[s]; c0 < end; c0 += chunk) {
            int32_t al[ITEMS];
#pragma unroll
            for (int k = 0; k < ITEMS; ++k) {
                const int32_t i = c0 + lbase + k * 64;
                al[k] = i < end ? v.al[s][i] : 1;
            }
            bool fr[ITEMS];
#pragma unroll
            for (int k = 0; k < ITEMS; ++k) {
                const int32_t i = c0 + lbase + k * 64;
                fr[k] = i < end && (al[k] == 0 || al[k] == 2);
            }
            uint32_t rank[ITEMS];
            const uint32_t tot = chunk_rank<ITEMS>(fr, rank, lds);
#pragma unroll
            for (int k = 0; k < ITEMS; ++k) {
                const int32_t i = c0 + lbase + k * 64;
                const uint32_t j = base_rank + rank[k];
                if (fr[k] && j < nb) {
                    int q = 0;   // the member whose list holds breeder j
                    while (q + 1 < tm.K && uint32_t(bpre[q + 1]) <= j) ++q;
                    const int32_t p = member_list(tm, q)[list_off + int32_t(j) - bpre[q]];
                    const int32_t ep = v.e[s][p];
                    const int32_t ec = ep >> 1;
                    v.x[s][i] = v.x[s][p];
                    v.y[s][i] = v.y[s][p];
                    v.e[s][i] = ec;
                    v.e[s][p] = ep - ec;
                    v.al[s][i] = 1;
                    top[s] = i + 1;
                    if (counts) atomicAdd(&counts->births[s], 1);
                } else if (i < end) {
                    // a breeder's energy stays positive, so no slot read by a child dies
                    // here, whichever of its two values another member's child leaves
                    const bool starves = al[k] != 0 && al[k] != 2 && v.e[s][i] < 0;
                    if (counts && starves) atomicAdd(&counts->starved[s], 1);
                    if (al[k] == 2 || starves)
                        v.al[s][i] = 0;
                    else if (al[k] != 0)
                        top[s] = i + 1;
                }
            }
            base_rank += tot;
        }
    }
    // the next step's marks (every wave is past its loops: the reduction's
    // first barrier comes after them)
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const int32_t m = block_max32(top[s], lds);
        if (threadIdx.x == 0) tm.s_mark[s] = m;
    }
    // births, deaths and re-armed claims are visible to the next step
    return team_sync(tm);
}

__device__ __forceinline__ void set_tags(ModelView& v, int64_t max_cap) {
    // claim keys: slots below 2^sb (caps are at most 2^30), a tag of up to
    // kTagBits bits above the 32-bit draw; tags tag_top down to 1 (0 alone when
    // one tag bit is left, re-arming every step); all-ones has a tag no step uses
    uint32_t sb = 1;
    while (sb < 31 && (int64_t(1) << sb) < max_cap) ++sb;
    const uint32_t tag_bits = 32 - sb < kTagBits ? 32 - sb : kTagBits;
    const uint64_t t_max = (uint64_t(1) << tag_bits) - 1;
    v.sb = sb;
    v.tag_top = t_max > 1 ? t_max - 1 : 0;
    v.period = t_max > 1 ? uint32_t(t_max - 1) : 1u;
    v.tag_mask = ~uint64_t(0) << (32 + sb);
}

__device__ ModelView view_of(const BatchArgs& a, const abm_model_desc* d) {
    ModelView v;
    v.W = d->W;
    v.H = d->H;
    v.R = d->R;
    v.gain[0] = d->gain_s;
    v.gain[1] = d->gain_w;
    v.T[0] = d->T_s;
    v.T[1] = d->T_w;
    v.seed = d->seed;
    v.multi = d->multi_prey != 0;
    set_tags(v, d->cap_s > d->cap_w ? d->cap_s : d->cap_w);
    v.link[0] = a.link_s ? a.link_s + d->sheep_off : nullptr;
    v.link[1] = a.link_w ? a.link_w + d->wolf_off : nullptr;
    v.cap[0] = int32_t(d->cap_s);
    v.cap[1] = int32_t(d->cap_w);
    v.ready = a.ready + d->cell_off;
    v.base = 0;
    v.claims = a.claims + 3 * d->cell_off;
    v.x[0] = a.sx + d->sheep_off;
    v.y[0] = a.sy + d->sheep_off;
    v.e[0] = a.se + d->sheep_off;
    v.al[0] = a.sa + d->sheep_off;
    v.x[1] = a.wx + d->wolf_off;
    v.y[1] = a.wy + d->wolf_off;
    v.e[1] = a.we + d->wolf_off;
    v.al[1] = a.wa + d->wolf_off;
    return v;
}

// Member ranges of a team for one launch, balanced by work: the members count
// the live agents of every 4096-slot block of their share of the model, and
// then every member computes the same bounds from the block costs (a slot
// costs 1 and a live agent 3 more: a dead slot is one coalesced load per pass,
// a live agent a draw, several gathers and atomics).  The live agents sit in
// the lowest slots (children take the lowest free slots), so equal slot
// counts would leave a few members with all the work.  False if a team barrier
// failed.
constexpr int32_t kBalBlock = 4096;

template <int ITEMS>
__device__ bool balance_team(const ModelView& v, Team& tm, uint32_t* lds) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int32_t chunk = int32_t(blockDim.x) * ITEMS;
    const int32_t lbase = wave * ITEMS * 64 + lane;
    int32_t* cost = member_list(tm, 0);   // lists are idle until the first step
    int32_t nblk[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) nblk[s] = (v.cap[s] + kBalBlock - 1) / kBalBlock;
    // live agents per block, each member over its share of the blocks
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const int32_t per = (nblk[s] + tm.K - 1) / tm.K;
        const int32_t b0 = min(nblk[s], tm.r * per), b1 = min(nblk[s], b0 + per);
        for (int32_t blk = b0; blk < b1; ++blk) {
            const int32_t lo = blk * kBalBlock, hi = min(v.cap[s], lo + kBalBlock);
            uint32_t live = 0;
            for (int32_t c0 = lo; c0 < hi; c0 += chunk) {
#pragma unroll
                for (int k = 0; k < ITEMS; ++k) {
                    const int32_t i = c0 + lbase + k * 64;
                    live += (i < hi && v.al[s][i] != 0) ? 1u : 0u;
                }
            }
            live = block_sum32(live, lds);
            if (threadIdx.x == 0) cost[(s ? nblk[0] : 0) + blk] = (hi - lo) + 3 * int32_t(live);
        }
    }
    if (!team_sync(tm)) return false;
    // bounds: member r starts at the first block whose cost prefix reaches
    // r / K of the total
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const int32_t* c = cost + (s ? nblk[0] : 0);
        int32_t* bound = tm.s_bound + s * (kMaxTeam + 1);
        uint32_t total = 0;
        for (int32_t b = threadIdx.x; b < nblk[s]; b += blockDim.x) total += uint32_t(c[b]);
        total = block_sum32(total, lds);
        if (threadIdx.x <= tm.K) bound[threadIdx.x] = threadIdx.x == 0 ? 0 : v.cap[s];
        __syncthreads();
        uint32_t carry = 0;
        for (int32_t b0 = 0; b0 < nblk[s]; b0 += int32_t(blockDim.x)) {
            const int32_t b = b0 + int32_t(threadIdx.x);
            const uint32_t mine = b < nblk[s] ? uint32_t(c[b]) : 0u;
            uint32_t incl;
            const uint32_t chunk_total = block_incl_scan32(mine, lds, &incl);
            const uint32_t before = carry + incl - mine;
            // the block where the prefix first reaches r * total / K
            for (int r = 1; r < tm.K; ++r) {
                const uint64_t target = (uint64_t(total) * uint32_t(r) + uint32_t(tm.K) - 1) /
                                        uint32_t(tm.K);
                if (b < nblk[s] && before < target && target <= before + mine)
                    bound[r] = min(v.cap[s], (b + 1) * kBalBlock);
            }
            carry += chunk_total;
        }
        __syncthreads();
        // bounds must not decrease (empty members keep a zero-width range)
        if (threadIdx.x == 0)
            for (int r = 1; r <= tm.K; ++r) bound[r] = max(bound[r], bound[r - 1]);
        __syncthreads();
    }
    return true;
}

// Runs model m's pending steps (at most `max_steps`) with team tm; member 0
// updates the descriptor.  A model of a single workgroup (no team) keeps its
// claim table in LDS when its 3 W H words fit in a.lds_words.  False if a
// team barrier failed.
template <int ITEMS>
__device__ bool run_model(const BatchArgs& a, int32_t m, int32_t max_steps, Team& tm,
                          uint32_t* lds) {
    abm_model_desc* d = a.models + m;
    if (d->cap_s + d->cap_w > a.scratch_stride || (d->multi_prey && !(a.link_s && a.link_w))) {
        // the descriptor does not fit the breeder list (max_cap too small), or
        // a multi-prey model has no list links: leave the model untouched and
        // report it
        if (threadIdx.x == 0 && tm.r == 0) st_agent(tm.err, 1ull);
        return true;
    }
    const ModelView v = view_of(a, d);
    const int32_t t0 = d->step;
    int32_t t1 = d->steps_target;
    if (t1 - t0 > max_steps) t1 = t0 + max_steps;
    if (tm.K > 1 && t1 > t0 && !balance_team<ITEMS>(v, tm, lds)) return false;
    uint64_t updates = 0;
    const bool local = tm.K == 1 && 3 * int64_t(v.W) * v.H <= a.lds_words;
    if (local && t1 > t0) local_fill(local_claims(), 3 * v.W * v.H);
    // no mark yet: the first step of the launch visits the whole range
    if (threadIdx.x == 0) {
        tm.s_mark[0] = INT32_MAX;
        tm.s_mark[1] = INT32_MAX;
    }
    __syncthreads();
    for (int32_t t = t0; t < t1; ++t) {
        uint32_t live;
        const bool last = t + 1 == t1;
        const bool ok =
            local ? model_step<ITEMS, true>(v, uint32_t(t), uint32_t(t0), last, tm, lds, &live)
                  : model_step<ITEMS, false>(v, uint32_t(t), uint32_t(t0), last, tm, lds, &live);
        if (!ok) return false;
        updates += live;
    }
    if (threadIdx.x == 0 && tm.r == 0 && t1 > t0) {
        d->step = t1;
        d->updates += int64_t(updates);
    }
    return true;
}

// Workgroups [0, team_wgs) form teams of team_k members and take models
// order[0, n_team) from queue 0; once that queue is empty they work alone like
// the other workgroups, which take order[n_team, n_models) from queue 1.
template <int ITEMS>
__global__ __launch_bounds__(1024) void k_batched_run(BatchArgs a) {
    __shared__ uint32_t lds[16];
    __shared__ int32_t s_pre[2 * (kMaxTeam + 1) + 3];
    __shared__ int32_t s_ok, s_model, s_steps;
    __shared__ int32_t s_bound[2 * (kMaxTeam + 1)];
    __shared__ int32_t s_mark[2];
    const uint32_t b = blockIdx.x;
    Team tm;
    tm.gen = 0;
    tm.scratch = a.scratch;
    tm.stride = a.scratch_stride;
    tm.counts = a.team_counts;
    tm.err = a.err;
    tm.s_pre = s_pre;
    tm.s_ok = &s_ok;
    tm.s_bound = s_bound;
    tm.s_mark = s_mark;
    if (b < a.team_wgs) {
        const uint32_t xcd = b % 8, idx = b / 8;
        const uint32_t team = xcd + 8 * (idx / a.team_k);
        tm.K = int(a.team_k);
        tm.r = int(idx % a.team_k);
        tm.base = xcd + 8 * (idx - uint32_t(tm.r));
        tm.ctr = a.team_ctr + team;
        int32_t* mailbox = a.team_mail + team;
        for (;;) {
            if (threadIdx.x == 0 && tm.r == 0) {
                const uint32_t q = atomicAdd(a.queue + kQueueTeam, 1u);
                __hip_atomic_store(mailbox, q < uint32_t(a.n_team) ? a.order[q] : -1,
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            if (!team_sync(tm)) return;
            if (threadIdx.x == 0)
                s_model = __hip_atomic_load(mailbox, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            // every member has read the mailbox before the leader writes it again
            if (!team_sync(tm)) return;
            const int32_t m = s_model;
            // every wave has read s_model before thread 0 reuses it (the solo
            // loop below writes it straight away)
            __syncthreads();
            if (m < 0) break;
            if (!run_model<ITEMS>(a, m, a.max_steps, tm, lds)) return;
            __syncthreads();   // (thread 0 rejoins its wave: see k_batched_chip)
        }
    }
    tm.K = 1;
    tm.r = 0;
    tm.base = b;
    tm.ctr = nullptr;
    for (;;) {
        if (threadIdx.x == 0) {
            if (a.listed) {
                const uint32_t n = a.queue[kSoloModels];
                const uint32_t q = n > 0 ? atomicAdd(a.queue + kQueueSolo, 1u) : 0u;
                const int64_t entry = q < n ? a.models[q].live_w : -1;
                s_model = int32_t(entry);
                s_steps = int32_t(entry >> 32);
            } else {
                const uint32_t q = uint32_t(a.n_team) + atomicAdd(a.queue + kQueueSolo, 1u);
                s_model = q < uint32_t(a.n_models) ? a.order[q] : -1;
                s_steps = a.max_steps;
            }
        }
        __syncthreads();
        const int32_t m = s_model, steps = s_steps;
        __syncthreads();
        if (m < 0) break;
        run_model<ITEMS>(a, m, steps, tm, lds);
        __syncthreads();   // (thread 0 rejoins its wave: see k_batched_chip)
    }
}

// Whether a model of n0 agents at the start is tried on the chip by workgroups
// of T threads.  Classes but the last (spare: half as many agents again) are
// left by the models that outgrow them for the next one.
template <int T>
__device__ __forceinline__ bool chip_room(int64_t bytes, int64_t cells, int64_t n0, bool spare) {
    int64_t rows = (bytes - chip_fixed_bytes<T>(cells)) / chip_row_bytes<int16_t>();
    rows = rows < ChipSize<T>::kMaxRows ? rows : ChipSize<T>::kMaxRows;
    return rows >= 2 && rows * 64 >= (spare ? n0 * 3 / 2 + 128 : n0 * 9 / 8);
}

// Entry k of a chip class's list, or of the list of the others.  (The
// descriptors' live counts are written when the run ends; until then they hold
// the lists of the last class, live_s, and of the others, live_w.)
__device__ __forceinline__ int64_t& chip_entry(const BatchArgs& a, int c, uint32_t k) {
    return c == kChipClasses - 1 ? a.models[k].live_s : a.chip_list[c][k];
}

// Sums of the sizes (cells plus slots) of the models on the chip and of the
// others, and the largest of each.
struct Sizes {
    uint64_t sum[2] = {0, 0}, most[2] = {0, 0};   // on the chip, others

    __device__ __forceinline__ void add(bool other, uint64_t size) {
        sum[other] += size;
        most[other] = size > most[other] ? size : most[other];
    }

    // ... over the workgroup of 1024 threads.
    __device__ __forceinline__ void reduce() {
        __shared__ uint64_t s_sum[2][16], s_most[2][16];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
#pragma unroll
            for (int o = 32; o >= 1; o >>= 1) {
                sum[k] += __shfl_xor((unsigned long long)sum[k], o, 64);
                const uint64_t x = __shfl_xor((unsigned long long)most[k], o, 64);
                most[k] = x > most[k] ? x : most[k];
            }
            if ((threadIdx.x & 63) == 0) {
                s_sum[k][threadIdx.x >> 6] = sum[k];
                s_most[k][threadIdx.x >> 6] = most[k];
            }
        }
        __syncthreads();
        *this = Sizes();
        for (int w = 0; w < 16; ++w)
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                sum[k] += s_sum[k][w];
                most[k] = s_most[k][w] > most[k] ? s_most[k][w] : most[k];
            }
    }

    // The chip launches run before the launch of the models that do not fit
    // them, so a batch with such models takes the sum of the two.  One launch of
    // all, a workgroup each, takes the time of its largest model, or that of all
    // sizes at the rate of some 56 models side by side; the chip takes a sixth
    // of it for its models.  Whichever is less, x 20 steps, in ms, one launch
    // against two: 40 models of 32^2 to 260^2 cells 1.94 and 2.23, 20 of 250^2 and
    // one of 270^2 2.07 and 2.31, 300 of 32^2 to 300^2, logarithmic, 3.0 and 3.2;
    // 200 of 250^2 and one of 400^2 6.5 and 4.6, 1000 of 32^2 to 260^2 6.4 and 3.6.
    __device__ __forceinline__ bool one_launch() const {
        constexpr uint64_t kSideBySide = 56, kChipGain = 6;
        const uint64_t others = sum[1] > kSideBySide * most[1] ? sum[1] : kSideBySide * most[1];
        return kChipGain * (sum[0] + sum[1]) < kChipGain * others + sum[0] + kSideBySide * most[0];
    }
};

// The models of one workgroup with steps to do, in launch order, as lists of
// model | steps << 32: one per chip class, and the others.  One workgroup.
__global__ __launch_bounds__(1024) void k_classify(BatchArgs a) {
    constexpr int kLists = kChipClasses + 1;
    __shared__ uint32_t s_cnt[kLists][16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    // list of the model at position i of the order (-1: none), its index and size
    const auto list_of = [&](int32_t i, int32_t* m, uint64_t* size) {
        *m = a.order[i];
        const abm_model_desc& d = a.models[*m];
        const int64_t cells = int64_t(d.W) * d.H, n0 = d.n_s0 + d.n_w0;
        const bool held = !d.multi_prey && d.W >= 1 && d.H >= 1 && d.W <= kChipSide &&
                          d.H <= kChipSide && d.R >= 1 && d.R <= kChipMaxR && d.gain_s >= 0 &&
                          d.gain_w >= 0 && d.gain_s <= kChipMaxGain &&
                          d.gain_w <= kChipMaxGain && d.cap_s + d.cap_w <= a.scratch_stride;
        int32_t list = kChipClasses;
        if (held && chip_room<256>(a.chip_bytes[0], cells, n0, true))
            list = 0;
        else if (held && chip_room<512>(a.chip_bytes[1], cells, n0, true))
            list = 1;
        else if (held && chip_room<1024>(a.chip_bytes[2], cells, n0, false))
            list = 2;
        if (d.steps_target <= d.step) list = -1;
        *size = uint64_t(cells + d.cap_s + d.cap_w);
        if (i < a.n_wide) {
            const bool wide = list == kChipClasses && int64_t(*size) >= kWideSize &&
                              d.cap_s + d.cap_w <= a.scratch_stride &&
                              (!d.multi_prey || (a.link_s && a.link_w));
            a.wide[i] = wide;
            if (wide) list = -1;
        }
        return list;
    };
    // (a batch of one round is looked at once)
    const bool once = a.n_models - a.n_team <= 1024;
    Sizes sizes;
    for (int32_t i = a.n_team + int32_t(threadIdx.x); i < a.n_models && !once; i += 1024) {
        int32_t m;
        uint64_t size;
        const int32_t list = list_of(i, &m, &size);
        if (list >= 0) sizes.add(list == kChipClasses, size);
    }
    bool one_launch = false;
    uint32_t n[kLists] = {};
    for (int32_t i0 = a.n_team; i0 < a.n_models; i0 += 1024) {
        const int32_t i = i0 + int32_t(threadIdx.x);
        int32_t m = 0, list = -1;
        uint64_t size = 0;
        if (i < a.n_models) list = list_of(i, &m, &size);
        if (i0 == a.n_team) {
            if (once && list >= 0) sizes.add(list == kChipClasses, size);
            if (__syncthreads_or(sizes.most[1] != 0)) {
                sizes.reduce();
                one_launch = sizes.one_launch();
            }
        }
        if (one_launch && list >= 0) list = kChipClasses;
        uint64_t b[kLists];
#pragma unroll
        for (int k = 0; k < kLists; ++k) b[k] = __ballot(list == k);
        __syncthreads();
        if (lane == 0)
#pragma unroll
            for (int k = 0; k < kLists; ++k) s_cnt[k][wave] = uint32_t(__popcll(b[k]));
        __syncthreads();
        const int64_t entry = (int64_t(a.max_steps) << 32) | m;
#pragma unroll
        for (int k = 0; k < kLists; ++k) {
            uint32_t at = n[k];
            for (int w = 0; w < wave; ++w) at += s_cnt[k][w];
            for (int w = 0; w < 16; ++w) n[k] += s_cnt[k][w];
            at += lane_rank(b[k]);
            if (list == k) {
                if (k < kChipClasses)
                    chip_entry(a, k, at) = entry;
                else
                    a.models[at].live_w = entry;
            }
        }
    }
    if (threadIdx.x == 0) {
#pragma unroll
        for (int k = 0; k < kChipClasses; ++k) a.queue[kChipModels + k] = n[k];
        a.queue[kSoloModels] = n[kChipClasses];
    }
}

// Models on the chip: one workgroup of T threads per model, class C.  A model
// that does not fit, or outgrows its class, goes (on) to the list of the next,
// and from the last one to that of the others.
template <int T, int C>
__global__ __launch_bounds__(T) void k_batched_chip(BatchArgs a) {
    extern __shared__ uint4 chip_lds[];
    __shared__ ChipShared sh;
    __shared__ int32_t s_model, s_steps;
    for (;;) {
        if (threadIdx.x == 0) {
            const uint32_t q = atomicAdd(a.queue + kQueueChip + C, 1u);
            const int64_t entry = q < a.queue[kChipModels + C] ? chip_entry(a, C, q) : -1;
            s_model = int32_t(entry);
            s_steps = int32_t(entry >> 32);
        }
        __syncthreads();
        const int32_t m = s_model, steps = s_steps;
        __syncthreads();
        if (m < 0) return;
        abm_model_desc* d = a.models + m;
        const ModelView v = view_of(a, d);
        const int32_t t0 = d->step;
        const int32_t t1 = d->steps_target - t0 > steps ? t0 + steps : d->steps_target;
        ChipStats st = {nullptr, 0};
        const int32_t t = run_on_chip<T, int16_t, false>(
            v, sh, reinterpret_cast<char*>(chip_lds), a.chip_bytes[C],
            a.scratch + int64_t(blockIdx.x) * a.scratch_stride, t0, t1, &st);
        if (threadIdx.x == ChipSize<T>::kKeeper) {
            d->step = t;
            d->updates += int64_t(st.updates);
            if (t < t1) {
                const int64_t entry = (int64_t(t1 - t) << 32) | m;
                if constexpr (C + 1 < kChipClasses)
                    chip_entry(a, C + 1, atomicAdd(a.queue + kChipModels + C + 1, 1u)) = entry;
                else
                    a.models[atomicAdd(a.queue + kSoloModels, 1u)].live_w = entry;
            }
        }
        // (without it the compiler may join this branch to the one the loop begins
        // with and run a lane apart from its wave's others, which then read the
        // last model again, without end)
        __syncthreads();
    }
}

// One small model (the one-model call): its grass as countdowns, statistics
// rows per step.
struct SmallArgs {
    int32_t W, H, R, gain[2];
    uint32_t T[2], seed;
    int32_t cap[2];
    int32_t* grass;
    uint64_t* claims;
    int32_t *x[2], *y[2], *e[2], *al[2];
    int32_t* scratch;          // cap[0] + cap[1] ints
    uint64_t* err;
    int64_t* stats;            // [n_steps][8] or null
    int32_t t0, n_steps, chip_bytes;
};

// The whole call in one workgroup, on the chip.  A state with live agents off the
// grid, which no run of this library leaves and the chip form does not hold, is
// stepped in global memory instead, as a batch's model of one workgroup is: 64 x
// 64 cells x 20 steps 0.30 ms (on the chip 0.13), 170 x 170 cells 0.77 (0.23).
__global__ __launch_bounds__(kChipThreads) void k_predation_small(SmallArgs a) {
    extern __shared__ uint4 chip_lds[];
    __shared__ ChipShared sh;
    __shared__ StepCounts counts;
    __shared__ uint32_t lds[16];
    __shared__ int32_t s_pre[2 * 2 + 3], s_mark[2];
    ModelView v;
    v.W = a.W;
    v.H = a.H;
    v.R = a.R;
    v.seed = a.seed;
    v.multi = false;
    v.ready = a.grass;
    v.claims = a.claims;
    for (int s = 0; s < 2; ++s) {
        v.gain[s] = a.gain[s];
        v.T[s] = a.T[s];
        v.cap[s] = a.cap[s];
        v.link[s] = nullptr;
        v.x[s] = a.x[s];
        v.y[s] = a.y[s];
        v.e[s] = a.e[s];
        v.al[s] = a.al[s];
    }
    set_tags(v, a.cap[0] > a.cap[1] ? a.cap[0] : a.cap[1]);
    const int32_t t1 = a.t0 + a.n_steps;
    ChipStats st = {a.stats, 0};
    const int32_t t = run_on_chip<kChipThreads, int32_t, true>(v, sh, reinterpret_cast<char*>(chip_lds),
                                                 a.chip_bytes, a.scratch, a.t0, t1, &st);
    if (t == t1) return;
    const int64_t cells = int64_t(a.W) * a.H;
    for (int64_t w = threadIdx.x; w < 3 * cells; w += blockDim.x) rearm(v.claims + w);
    v.base = t;               // the countdowns as they are: no sum that could overflow
    Team tm = {};
    tm.K = 1;
    tm.scratch = a.scratch;
    tm.err = a.err;
    tm.s_pre = s_pre;
    tm.s_mark = s_mark;
    if (threadIdx.x < 2) s_mark[threadIdx.x] = INT32_MAX;
    __builtin_amdgcn_s_waitcnt(0);
    for (int32_t k = t; k < t1; ++k) {
        if (threadIdx.x == 0) counts = StepCounts{};
        __syncthreads();
        uint32_t live;
        model_step<1, false>(v, uint32_t(k), uint32_t(t), k + 1 == t1, tm, lds, &live, &counts);
        if (threadIdx.x == 0 && a.stats) {
            int64_t* r = a.stats + 8 * int64_t(k - a.t0);
            r[0] = counts.live[0];
            r[1] = counts.live[1];
            r[2] = counts.grass;
            r[3] = counts.eaten;
            r[4] = counts.births[0];
            r[5] = counts.births[1];
            r[6] = counts.starved[0];
            r[7] = counts.starved[1];
        }
        __syncthreads();
    }
    for (int64_t c = threadIdx.x; c < cells; c += blockDim.x) {
        const int64_t d = int64_t(v.ready[c]) - (t1 - t);
        v.ready[c] = d > 0 ? int32_t(d) : 0;
    }
}

// Workgroups of the kernels that stream every model once, shared evenly (the
// host does not know the sizes): 64 a model, as there were, cost their dispatch
// where models are many and small (init of 2000 models of 32^2 to 64^2 cells
// 131 to 42 us; with 65536 workgroups 103, with 8192 36) and were few for one
// large model (1024^2: 53 to 18 us).
constexpr int32_t kModelBlocks = 16384;

// Elements of `size` bytes from the start of a 128-byte line to offset o.  The
// workgroups of a model lie on different XCDs, whose L2s each write their part
// of a line that two of them share; started at a line's start, they share none
// (init of 4096 models of 32^2 to 256^2 cells, 3.65 GB: 1275 to 739 us, 4.9
// TB/s).  An array that does not start at a line's start is only slower.
__device__ __forceinline__ int64_t line_skew(int64_t o, int size) {
    return o & (128 / size - 1);
}

// Initial state of every model (same definition as the one-model path), bound by
// the bytes written.
__global__ __launch_bounds__(256) void k_batched_init(abm_model_desc* models, int32_t n_models,
                                                     int32_t* ready, uint64_t* claims,
                                                     int32_t* sx, int32_t* sy, int32_t* se,
                                                     int32_t* sa, int32_t* wx, int32_t* wy,
                                                     int32_t* we, int32_t* wa) {
    const abm_model_desc& d = models[blockIdx.y];
    const int64_t G = int64_t(d.W) * d.H;
    const uint64_t key = stream_key(d.seed, kInitStep);
    const int64_t first = int64_t(blockIdx.x) * 256 + threadIdx.x, stride = int64_t(gridDim.x) * 256;
    for (int64_t i = first - line_skew(d.cell_off, 4); i < G; i += stride) {
        if (i < 0) continue;
        const uint32_t h = draw(key, uint32_t(i), kGrassGrown);
        ready[d.cell_off + i] =
            h < 0x80000000u
                ? 0
                : 1 + int32_t(scale(draw(key, uint32_t(i), kGrassCountdown), uint32_t(d.R)));
    }
    uint64_t* cw = claims + 3 * d.cell_off;
    for (int64_t i = first - line_skew(3 * d.cell_off, 8); i < 3 * G; i += stride)
        if (i >= 0) cw[i] = kNoClaim;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const int64_t cap = s ? d.cap_w : d.cap_s;
        const int64_t n0 = s ? d.n_w0 : d.n_s0;
        const int32_t gain = s ? d.gain_w : d.gain_s;
        const uint32_t px = s ? kWolfX : kSheepX;
        const int64_t o = s ? d.wolf_off : d.sheep_off;
        int32_t* X = (s ? wx : sx) + o;
        int32_t* Y = (s ? wy : sy) + o;
        int32_t* E = (s ? we : se) + o;
        int32_t* A = (s ? wa : sa) + o;
        for (int64_t i = first - line_skew(o, 4); i < cap; i += stride) {
            if (i < 0) continue;
            int32_t x = 0, y = 0, e = 0, al = 0;
            if (i < n0) {
                x = int32_t(scale(draw(key, uint32_t(i), px), uint32_t(d.W)));
                y = int32_t(scale(draw(key, uint32_t(i), px + 1), uint32_t(d.H)));
                e = int32_t(scale(draw(key, uint32_t(i), px + 2), uint32_t(2 * gain)));
                al = 1;
            }
            X[i] = x;
            Y[i] = y;
            E[i] = e;
            A[i] = al;
        }
    }
}

// countdown[c] = max(0, ready[c] - step) for every cell of every model.
__global__ __launch_bounds__(256) void k_batched_grass(const abm_model_desc* models,
                                                      const int32_t* ready, int32_t* countdown) {
    const abm_model_desc& d = models[blockIdx.y];
    const int64_t G = int64_t(d.W) * d.H;
    for (int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x - line_skew(d.cell_off, 4); i < G;
         i += int64_t(gridDim.x) * 256) {
        if (i < 0) continue;
        const int32_t r = ready[d.cell_off + i] - d.step;
        countdown[d.cell_off + i] = r > 0 ? r : 0;
    }
}

// Live counts per model (stored into the descriptors): eight loads of a thread
// in flight (96 models of up to 1002^2 cells: 700 us one at a time, by 256
// threads each; 57 so with 1024, 114 with 256).  Models of up to kCountFew slots
// a species have 256 threads, as many small workgroups are dispatched sooner
// (4096 models of 32^2 to 64^2 cells 28.6 to 9.3 us, of 32^2 to 200^2 39.6 to 24.6;
// eight of 256^2, past it, 4.8 with 1024 and 8.6 with 256).
constexpr int kCountAhead = 8;
constexpr int64_t kCountFew = 1 << 14;

template <int T>
__device__ __forceinline__ uint32_t count_live(const int32_t* alive, int64_t cap) {
    uint32_t n = 0;
    for (int64_t i0 = threadIdx.x; i0 < cap; i0 += T * kCountAhead) {
        int32_t v[kCountAhead];
#pragma unroll
        for (int k = 0; k < kCountAhead; ++k) {
            const int64_t i = i0 + k * T;
            v[k] = alive[i < cap ? i : i0];
        }
#pragma unroll
        for (int k = 0; k < kCountAhead; ++k) n += v[k] != 0 && i0 + k * T < cap;
    }
    return n;
}

template <int T>
__global__ __launch_bounds__(T) void k_batched_count(abm_model_desc* models, const int32_t* sa,
                                                     const int32_t* wa) {
    __shared__ uint32_t lds[T / 64];
    abm_model_desc& d = models[blockIdx.x];
    const uint32_t ls = block_sum32(count_live<T>(sa + d.sheep_off, d.cap_s), lds);
    const uint32_t lw = block_sum32(count_live<T>(wa + d.wolf_off, d.cap_w), lds);
    if (threadIdx.x == 0) {
        d.live_s = ls;
        d.live_w = lw;
    }
}

// Clears the queue counters and the team barrier counters of a run.
__global__ void k_reset_queue(uint32_t* q, uint32_t* team_ctr, int32_t n_teams) {
    const int32_t i = blockIdx.x * 256 + threadIdx.x;
    if (i < kQueueWords) q[i] = 0;
    if (i < n_teams) team_ctr[i] = 0;
}

int check_batch(const abm_batch* b) {
    if (!b) return fail(ABM_E_INVALID, "batch is NULL");
    if (b->n_models < 0 || b->n_models > 65535)
        return fail(ABM_E_INVALID, "n_models must be in [0, 65535]");
    if (b->n_models == 0) return ABM_OK;
    if (!b->models || !b->ready || !b->claims) return fail(ABM_E_INVALID, "batch array is NULL");
    const abm_species* sp[2] = {&b->sheep, &b->wolves};
    for (int k = 0; k < 2; ++k)
        if (!sp[k]->x || !sp[k]->y || !sp[k]->e || !sp[k]->alive)
            return fail(ABM_E_INVALID, "species array is NULL");
    if (b->max_cap < 1 || b->max_cap > (1 << 30))
        return fail(ABM_E_INVALID, "max_cap must be in [1, 2^30]");
    return ABM_OK;
}

}  // namespace
}  // namespace abm

using namespace abm;

// Workspace of a batched run: a 256-byte header (queue counters; error word at
// byte 248), the team area (barrier counter and model mailbox per team, member
// counts per workgroup) and one breeder list (2 * max_cap ints) per workgroup.
constexpr int64_t kTeamAreaWords = int64_t(kMaxWorkgroups) * (2 + kCountWords);
// The count words of the team area hold a byte per wide model and two lists of
// models on the chip when no team runs.
constexpr int kMaxWideModels = kMaxWorkgroups;
constexpr int64_t kChipListed = 9000;
// Models times steps of a run from which four small models share a CU, and the
// capacity up to which a step or two of many models are left to one launch (see
// abm_predation_run_batched).
constexpr int64_t kFourWork = 24000;
constexpr int64_t kTinyCap = 4096;
static_assert(2 * kMaxWideModels + 64 + 16 * kChipListed <=
                  4 * int64_t(kMaxWorkgroups) * kCountWords, "the lists fit the count words");

extern "C" size_t abm_batched_workspace_bytes(int64_t max_cap, int32_t n_workgroups) {
    if (max_cap < 1 || max_cap > (int64_t(1) << 30) || n_workgroups < 1 ||
        n_workgroups > kMaxWorkgroups)
        return 0;
    return size_t(kHeaderBytes) + size_t(4 * kTeamAreaWords) +
           size_t(n_workgroups) * size_t(2 * max_cap) * 4 + 256;
}

namespace {

uint32_t model_blocks(int32_t n_models) {
    const int32_t k = kModelBlocks / n_models;
    return uint32_t(k < 4 ? 4 : (k > 256 ? 256 : k));
}

}  // namespace

extern "C" int abm_predation_batched_init(const abm_batch* b, void* stream) {
    int rc = check_batch(b);
    if (rc != ABM_OK || b->n_models == 0) return rc;
    rc = check_device();
    if (rc != ABM_OK) return rc;
    const dim3 grid(model_blocks(b->n_models), static_cast<uint32_t>(b->n_models));
    hipLaunchKernelGGL(k_batched_init, grid, dim3(256), 0, as_stream(stream), b->models,
                       b->n_models, b->ready, b->claims, b->sheep.x, b->sheep.y, b->sheep.e,
                       b->sheep.alive, b->wolves.x, b->wolves.y, b->wolves.e, b->wolves.alive);
    return launch_status("predation_batched_init");
}

namespace {

const void* run_kernel(int items) {
    return items == 1 ? reinterpret_cast<const void*>(k_batched_run<1>)
         : items == 2 ? reinterpret_cast<const void*>(k_batched_run<2>)
                      : reinterpret_cast<const void*>(k_batched_run<4>);
}

// Launch shape of a run: workgroups resident per CU at `block` threads and
// the dynamic LDS each can hold without lowering that count (the CU's LDS
// shared among them, less the kernel's static LDS; at most the per-workgroup
// limit).  False with the error set if a query fails.
bool run_shape(int items, int block, int* n_cu, int* per_cu, int64_t* lds_bytes) {
    const void* kern = run_kernel(items);
    int dev = 0, lds_cu = 0, lds_block = 0;
    hipFuncAttributes fa;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipDeviceGetAttribute(&lds_cu, hipDeviceAttributeMaxSharedMemoryPerMultiprocessor,
                              dev) != hipSuccess ||
        hipDeviceGetAttribute(&lds_block, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) !=
            hipSuccess ||
        hipFuncGetAttributes(&fa, kern) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(per_cu, kern, block, 0) != hipSuccess) {
        set_error("predation_run_batched: device query failed");
        return false;
    }
    if (*per_cu < 1) *per_cu = 1;
    int64_t dyn = int64_t(lds_cu) / *per_cu - int64_t(fa.sharedSizeBytes);
    if (dyn > int64_t(lds_block) - int64_t(fa.sharedSizeBytes))
        dyn = int64_t(lds_block) - int64_t(fa.sharedSizeBytes);
    dyn = dyn > 0 ? dyn / 1024 * 1024 : 0;
    // allocation granularity: step down until the occupancy is unchanged
    for (; dyn > 0; dyn -= 1024) {
        int with = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&with, kern, block, size_t(dyn)) !=
            hipSuccess) {
            set_error("predation_run_batched: occupancy query failed");
            return false;
        }
        if (with >= *per_cu) break;
    }
    *lds_bytes = dyn;
    return true;
}

// Dynamic LDS a workgroup of the largest on-chip class can take on the current
// device (the per-workgroup limit less their static LDS), looked up once per
// device; 0 if a query fails.
constexpr int kChipDevices = 64;
std::atomic<int> g_chip_bytes[kChipDevices];

int chip_lds_bytes() {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kChipDevices) return 0;
    int n = g_chip_bytes[dev].load(std::memory_order_relaxed);
    if (n == 0) {
        int lds_block = 0;
        hipFuncAttributes fb, fs;
        if (hipDeviceGetAttribute(&lds_block, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) !=
                hipSuccess ||
            hipFuncGetAttributes(&fb, reinterpret_cast<const void*>(k_batched_chip<1024, 2>)) !=
                hipSuccess ||
            hipFuncGetAttributes(&fs, reinterpret_cast<const void*>(k_predation_small)) != hipSuccess)
            return 0;
        const size_t fixed = fb.sharedSizeBytes > fs.sharedSizeBytes ? fb.sharedSizeBytes : fs.sharedSizeBytes;
        n = (lds_block - int(fixed)) / 1024 * 1024;
        if (n < 1024) n = 1024;       // (holds no model)
        g_chip_bytes[dev].store(n, std::memory_order_relaxed);
    }
    return n;
}

// ... and of a class of which `per_cu` workgroups are to share a CU: its part,
// less the static LDS and an allocation unit.
int chip_lds_part(int whole, int per_cu) {
    const int n = (whole / per_cu - 2048) / 1024 * 1024;
    return n > 0 ? n : 0;
}

}  // namespace

namespace abm {

// A small model advanced by one workgroup on the chip: every slot of both
// species and every cell fit its LDS, so whatever the populations do the call
// is one launch.  20 steps from the initial state, in us, against the general
// path's launches: 64 x 64 cells with 511 agents 128 and 303, with 5120 248 and
// 480; 170 x 170 cells with 3612 agents 233 and 550, with 15104 557 and 567.
//   With many more slots than cells a first step can find several agents in
// every cell, which one workgroup is slow at (20000 agents on 64 x 64 cells: 183
// us against 53), so past 1.5 slots a cell only models of up to 1024 slots are
// taken.
//   A call of one step loads and stores the whole state for it: 28 against 37 us
// at 64 x 64 cells with 511 agents, 53 and 48 with 5120; 50 and 50 at 170 x 170
// with 3612, 107 and 52 with 15104.  The call does not know the number of
// agents, so a single step of more than kOneStepSlots slots is left to the
// launches, whose time hardly depends on it.
constexpr int64_t kOneStepSlots = 8192;

int launch_small_predation(const abm_predation_params* p, const abm_predation_state* s,
                           int32_t n_steps, const Workspace& w, hipStream_t st, bool* taken) {
    *taken = false;
    if (p->W > kChipSide || p->H > kChipSide || p->R > kChipMaxR || p->multi_prey ||
        uint64_t(s->step) + uint64_t(n_steps) > 0x7FFFFFFFull)
        return ABM_OK;
    const int64_t cells = int64_t(p->W) * p->H;
    const int64_t rows = tiles_for(p->cap_s, 64) + tiles_for(p->cap_w, 64);
    const int64_t need = chip_fixed_bytes<kChipThreads>(cells) + rows * chip_row_bytes<int32_t>();
    const int bytes = chip_lds_bytes();
    const int64_t slots = p->cap_s + p->cap_w;
    if (need > bytes || (slots > 1024 && 2 * slots > 3 * cells) ||
        (n_steps == 1 && slots > kOneStepSlots))
        return ABM_OK;
    SmallArgs a;
    a.W = p->W;
    a.H = p->H;
    a.R = p->R;
    a.gain[0] = p->gain_s;
    a.gain[1] = p->gain_w;
    a.T[0] = p->T_s;
    a.T[1] = p->T_w;
    a.seed = p->seed;
    a.cap[0] = int32_t(p->cap_s);
    a.cap[1] = int32_t(p->cap_w);
    a.grass = s->grass;
    a.claims = s->claims;
    const abm_species* sp[2] = {&s->sheep, &s->wolves};
    for (int k = 0; k < 2; ++k) {
        a.x[k] = sp[k]->x;
        a.y[k] = sp[k]->y;
        a.e[k] = sp[k]->e;
        a.al[k] = sp[k]->alive;
    }
    a.scratch = w.list_a;             // (both lists: twice the larger capacity)
    a.err = w.hdr + kHdrError;
    a.stats = s->stats;
    a.t0 = int32_t(s->step);
    a.n_steps = n_steps;
    a.chip_bytes = int32_t(need);
    hipLaunchKernelGGL(k_predation_small, dim3(1), dim3(kChipThreads), size_t(need), st, a);
    *taken = true;
    return launch_status("predation_step");
}

}  // namespace abm

extern "C" int64_t abm_batched_lds_cells(int32_t block_threads, int32_t items) {
    if (block_threads < 256 || block_threads > 1024 || (block_threads & 63)) return 0;
    if (items != 1 && items != 2 && items != 4) return 0;
    if (check_device() != ABM_OK) return 0;
    int n_cu = 0, per_cu = 0;
    int64_t lds_bytes = 0;
    if (!run_shape(items, block_threads, &n_cu, &per_cu, &lds_bytes)) return 0;
    return lds_bytes / 24;
}

extern "C" int abm_predation_run_batched(const abm_batch* b, const int32_t* order,
                                         int32_t max_steps, const abm_tuning* tune, void* ws,
                                         size_t ws_bytes, void* stream) {
    int rc = check_batch(b);
    if (rc != ABM_OK) return rc;
    if (max_steps < 0) return fail(ABM_E_INVALID, "max_steps must be >= 0");
    if (b->n_models == 0 || max_steps == 0) return ABM_OK;
    if (!order) return fail(ABM_E_INVALID, "order is NULL");
    rc = check_device();
    if (rc != ABM_OK) return rc;
    int block = tune && tune->block_threads ? tune->block_threads : 512;
    if (block < 256 || block > 1024 || (block & 63))
        return fail(ABM_E_INVALID, "block_threads must be a multiple of 64 in [256, 1024]");
    const int items = tune && tune->items ? tune->items : 4;
    if (items != 1 && items != 2 && items != 4)
        return fail(ABM_E_INVALID, "items must be 1, 2 or 4");
    int n_cu = 0, per_cu = 0;
    int64_t lds_bytes = 0;
    if (!run_shape(items, block, &n_cu, &per_cu, &lds_bytes)) return ABM_E_HIP;
    if (tune && tune->global_claims) lds_bytes = 0;
    int resident = n_cu * per_cu;
    const size_t fixed = size_t(abm_batched_workspace_bytes(b->max_cap, 1)) - size_t(8 * b->max_cap);
    const int64_t shares = ws_bytes > fixed ? int64_t((ws_bytes - fixed) / size_t(8 * b->max_cap)) : 0;
    // a caller that asks for fewer workgroups than would be resident and its
    // workspace has shares for leaves the rest of the device to others, whichever
    // kernels advance its models
    const bool bounded =
        tune && tune->workgroups > 0 && tune->workgroups < resident && tune->workgroups < shares;
    if (tune && tune->workgroups > 0 && tune->workgroups < resident) resident = tune->workgroups;
    if (resident > kMaxWorkgroups) resident = kMaxWorkgroups;
    // teams: order[0, n_team) is run by teams of K workgroups, formed from the
    // first team_wgs workgroups (a multiple of 8 K)
    const int K = tune && tune->team_size > 1 ? tune->team_size : 1;
    int n_team = K > 1 && tune ? tune->team_models : 0;
    if (K > kMaxTeam) return fail(ABM_E_INVALID, "team_size must be at most 16");
    if (n_team < 0 || n_team > b->n_models)
        return fail(ABM_E_INVALID, "team_models must be in [0, n_models]");
    int team_wgs = 0;
    if (n_team > 0) {
        const int unit = 8 * K;
        const int fit = resident / unit * unit;
        if (fit == 0) {
            set_error("teams of %d need %d resident workgroups, %d are available", K, unit,
                      resident);
            return ABM_E_INVALID;
        }
        team_wgs = tune->team_workgroups > 0 ? tune->team_workgroups
                                             : (n_team * K + unit - 1) / unit * unit;
        if (team_wgs % unit != 0)
            return fail(ABM_E_INVALID, "team_workgroups must be a multiple of 8 * team_size");
        if (team_wgs > fit) team_wgs = fit;
    }
    int grid = resident - team_wgs;
    if (grid > b->n_models - n_team) grid = b->n_models - n_team;
    grid += team_wgs;
    const size_t need = abm_batched_workspace_bytes(b->max_cap, grid);
    if (!ws || ws_bytes < need) {
        set_error("workspace has %zu bytes, needs %zu", ws_bytes, need);
        return ABM_E_WORKSPACE;
    }
    if ((reinterpret_cast<uintptr_t>(ws) & 255) != 0)
        return fail(ABM_E_WORKSPACE, "workspace must be 256-byte aligned");
    hipStream_t st = as_stream(stream);
    BatchArgs a;
    a.models = b->models;
    a.order = order;
    a.n_models = b->n_models;
    a.max_steps = max_steps;
    a.ready = b->ready;
    a.claims = b->claims;
    a.sx = b->sheep.x;
    a.sy = b->sheep.y;
    a.se = b->sheep.e;
    a.sa = b->sheep.alive;
    a.wx = b->wolves.x;
    a.wy = b->wolves.y;
    a.we = b->wolves.e;
    a.wa = b->wolves.alive;
    a.link_s = b->link_s;
    a.link_w = b->link_w;
    char* base = static_cast<char*>(ws);
    a.queue = reinterpret_cast<uint32_t*>(base);
    a.err = reinterpret_cast<uint64_t*>(base + kHeaderBytes - 8);
    a.team_ctr = reinterpret_cast<uint32_t*>(base + kHeaderBytes);
    a.team_mail = reinterpret_cast<int32_t*>(a.team_ctr + kMaxWorkgroups);
    a.team_counts = a.team_mail + kMaxWorkgroups;
    a.scratch = reinterpret_cast<int32_t*>(base + kHeaderBytes + 4 * kTeamAreaWords);
    a.scratch_stride = 2 * b->max_cap;
    a.n_team = n_team;
    a.lds_words = int32_t(lds_bytes / 8);
    // The models that would run in teams, and the largest of the others, by
    // launches over the whole device instead, all of them side by side, where
    // the workspace has two shares for each
    int n_wide = 0;
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (n_team > 0 && hipStreamIsCapturing(st, &capture) != hipSuccess)
        return fail(ABM_E_HIP, "hipStreamIsCapturing failed");
    const int32_t most = capture == hipStreamCaptureStatusNone ? kWideSteps : kWideStepsRecorded;
    if (n_team > 0 && !bounded && max_steps <= most && 2 * int64_t(n_team) <= shares &&
        n_team < kMaxWideModels && wide_fits(b->max_cap)) {
        // (the order is largest first where it balances the load)
        const int with = n_team + 8 < kWideAtLeast ? kWideAtLeast : n_team + 8;
        n_wide = b->n_models < with ? b->n_models : with;
        if (n_wide > shares / 2) n_wide = int(shares / 2);
        team_wgs = 0;
        grid = resident < b->n_models - n_team ? resident : b->n_models - n_team;
        if (grid > shares) grid = int(shares);
    }
    a.team_k = uint32_t(K);
    a.team_wgs = uint32_t(team_wgs);
    const int n_teams = team_wgs / K;
    hipLaunchKernelGGL(k_reset_queue, dim3((n_teams + 255) / 256 + 1), dim3(256), 0, st, a.queue,
                       a.team_ctr, n_teams);
    a.listed = 0;
    for (int c = 0; c < kChipClasses; ++c) {
        a.chip_bytes[c] = 0;
        a.chip_list[c] = nullptr;
    }
    // Models of one workgroup go to the chip (4096 models of 32^2 to 256^2 cells
    // x 50 steps: 50.4 to 7.5 ms), unless there are teams: they run in the time
    // those take anyway, and a launch before them only delays the teams.  A batch
    // with links holds models matched by rank, which do not go there; all of its
    // models run as one launch, since looking for others costs more than it may
    // find (1000 models of 32^2 to 64^2, all by rank, x 10 steps: 489 and 600 us).
    a.wide = reinterpret_cast<uint8_t*>(a.team_counts);
    a.n_wide = 0;
    const int bound = bounded ? resident : 4 * n_cu;   // workgroups of a chip launch
    const bool links = b->link_s && b->link_w;
    const int64_t solo = b->n_models - n_team;
    // One step of many tiny models does not repay the list and the launches (1000
    // of 32^2 to 64^2 cells, up to 1636 slots a species: 107 us in one launch, 125
    // with the chip; of 32^2 to 200^2, up to 16000: 342 and 144), and neither do two
    // of models that a round or two of workgroups hold (1000 of 24^2 to 40^2: 108 and
    // 118; 300 of 24^2 to 64^2 81 and 70, 2000 222 and 199)
    const bool tiny = solo > n_cu && b->max_cap <= kTinyCap &&
                      (max_steps == 1 || (max_steps == 2 && solo <= 4 * n_cu));
    const bool chips = !(tune && tune->global_claims) && team_wgs == 0 && solo > 0 &&
                       (n_wide > 0 || (!links && !tiny));
    if (chips) {
        const int chip = chip_lds_bytes();
        if (chip > 0) {
            a.listed = 1;
            a.n_wide = n_wide;
            a.chip_bytes[2] = chip;
            // The smaller classes put two or four models on a CU, which pays when
            // there are more models than CUs: a workgroup waits for the latency of
            // its parts, and another one's fill the gaps (x 50 steps, in ms: 4096
            // models of 32^2 to 64^2 cells 3.7 to 1.4, of 100^2 to 150^2 6.2 to 4.3,
            // of 32^2 to 256^2 8.5 to 7.7; 300 of 100^2 to 150^2 0.73 to 0.60).
            // Each is a launch of its own, so they need steps: 1000 models of 32^2 to
            // 64^2 x 1 step take 125, 138 and 205 us with one, two and three classes,
            // x 3 142, 140 and 199, x 10 295, 226 and 254, x 40 790, 498 and 403; 4096
            // of 24^2 to 64^2 x 8 two 496 and three 509, x 15 736 and 625.
            // Their lists lie behind the bytes of `wide`
            if (solo <= kChipListed && solo > n_cu && bound >= 2 * n_cu && max_steps > 1) {
                a.chip_list[1] = reinterpret_cast<int64_t*>(a.wide + 2 * kMaxWideModels + 64);
                a.chip_list[0] = a.chip_list[1] + kChipListed;
                a.chip_bytes[1] = chip_lds_part(chip, 2);
                if (solo > 2 * n_cu && bound >= 4 * n_cu && solo * max_steps >= kFourWork)
                    a.chip_bytes[0] = chip_lds_part(chip, 4);
            }
            hipLaunchKernelGGL(k_classify, dim3(1), dim3(1024), 0, st, a);
        }
    }
    if (n_wide > 0) {
        WideArgs w;
        w.models = b->models;
        w.order = order;
        w.ready = b->ready;
        w.claims = b->claims;
        w.sheep = b->sheep;
        w.wolves = b->wolves;
        w.link_s = b->link_s;
        w.link_w = b->link_w;
        w.err = a.err;
        w.taken = a.wide;
        w.count = a.queue + kWideModels;
        w.shares = reinterpret_cast<char*>(a.scratch);
        w.share = 8 * b->max_cap;
        w.max_cap = b->max_cap;
        w.n = a.listed ? n_wide : n_team;
        w.n_team = n_team;
        w.max_steps = max_steps;
        rc = launch_wide(w, st);
        if (rc != ABM_OK) return rc;
    }
    if (a.listed) {
        // (a share of the workspace each)
        const int room = solo < shares ? int(solo) : int(shares);
        const int most = room < bound ? room : bound;
        const auto wgs = [&](int per_cu) { return dim3(per_cu * n_cu < most ? per_cu * n_cu : most); };
        if (a.chip_bytes[0] > 0)
            hipLaunchKernelGGL((k_batched_chip<256, 0>), wgs(4), dim3(256),
                               size_t(a.chip_bytes[0]), st, a);
        if (a.chip_bytes[1] > 0)
            hipLaunchKernelGGL((k_batched_chip<512, 1>), wgs(2), dim3(512),
                               size_t(a.chip_bytes[1]), st, a);
        hipLaunchKernelGGL((k_batched_chip<1024, 2>), wgs(1), dim3(1024), size_t(a.chip_bytes[2]),
                           st, a);
    }
    const size_t dyn = size_t(lds_bytes);
    if (grid > 0) switch (items) {
        case 1: hipLaunchKernelGGL(k_batched_run<1>, dim3(grid), dim3(block), dyn, st, a); break;
        case 2: hipLaunchKernelGGL(k_batched_run<2>, dim3(grid), dim3(block), dyn, st, a); break;
        default: hipLaunchKernelGGL(k_batched_run<4>, dim3(grid), dim3(block), dyn, st, a); break;
    }
    if (b->max_cap <= kCountFew)
        hipLaunchKernelGGL(k_batched_count<256>, dim3(b->n_models), dim3(256), 0, st, b->models,
                           b->sheep.alive, b->wolves.alive);
    else
        hipLaunchKernelGGL(k_batched_count<1024>, dim3(b->n_models), dim3(1024), 0, st, b->models,
                           b->sheep.alive, b->wolves.alive);
    return launch_status("predation_run_batched");
}

extern "C" int abm_predation_batched_grass(const abm_batch* b, int32_t* countdown, void* stream) {
    int rc = check_batch(b);
    if (rc != ABM_OK || b->n_models == 0) return rc;
    if (!countdown) return fail(ABM_E_INVALID, "countdown is NULL");
    rc = check_device();
    if (rc != ABM_OK) return rc;
    const dim3 grid(model_blocks(b->n_models), static_cast<uint32_t>(b->n_models));
    hipLaunchKernelGGL(k_batched_grass, grid, dim3(256), 0, as_stream(stream), b->models, b->ready,
                       countdown);
    return launch_status("predation_batched_grass");
}
