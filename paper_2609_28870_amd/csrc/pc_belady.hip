// Belady's MIN at many cache capacities (pc_belady): the offline ceiling the
// paper compares every online policy with (Sec. 3.2 "Belady's optimum"),
// and the LRU-Belady gap under concurrency (Appendix B).
//
// Demand paging: every accessed block is brought in; when the cache is full
// the victim is the resident block whose next use is farthest away, a block
// that is never used again being farthest of all.  Only next[] is needed.
// Identify a resident block with its next-use position: the block accessed
// at t was inserted at prev(t) with value t, so the access at t hits exactly
// when value t is still present, and is then replaced by next(t).  Values
// are distinct positions (next is one-to-one), blocks without a next use are
// only counted ("dead"), and the victim is a dead block if there is one,
// else the largest value.  Victim ties exist only among dead blocks, so the
// hit count is unique.
//
// GPU mapping: one workgroup of one wave per capacity, all capacities at
// once; each wave runs its capacity's simulation through the trace, 64
// accesses (one per lane) at a time.  The values below a threshold theta
// are bits of a bitmap over positions; the values at or above it, the ones
// evictions take, sit in a sorted buffer in LDS (largest first).  The
// bitmap's words for the 4096 positions just past the batch live in an LDS
// ring, the rest in global memory (with a one-bit-per-word summary).
// Before a batch the buffer's values that fall inside its 64 positions
// leave it for a window register, so the values present in the window are
// that register and one ring word.  Blocks accessed earlier in the same
// batch come back inside it: their next uses are one-hot bits of the window.
//   * When the batch needs no eviction, or only as many as there are dead
//     blocks, nothing in the window can leave: the hits are the window word
//     or'ed with those bits (a wave OR), and the batch's inserts go to the
//     dead count, the bitmap or the buffer in bulk.
//   * Otherwise the evictions (after the dead blocks) take the largest
//     values present, which are among the buffer's top 64 and the batch's
//     own inserts above theta; the wave decides them all at once (a prefix
//     maximum finds the evictions, and each lane, for its own insert, whether
//     one of them takes it, from a walk over the batch, six accesses per entry
//     of a table in LDS).  Which inserts of its batch lie above an access's own
//     does not depend on the capacity: a kernel of its own finds that once, a
//     64-bit mask per access.  When those candidates run out the wave
//     walks the batch in access order instead, refilling the buffer from the
//     bitmap's largest values above the window (whole words, top down) and
//     taking the window's largest value when nothing above it is left.
// Values inserted above theta are merged into the buffer in sorted order
// after the batch; a buffer above 160 values spills its lowest into the
// bitmap.  Global bitmap words are touched only by their capacity's wave,
// through relaxed device-scope atomics (they live in L2).  A word entering
// the ring may still hold bits inserted before: every 16 batches, after a
// fence, the words that entered are exchanged for zero and their bits are
// merged into the ring at the next such sync, long before the window gets
// there, so a batch waits on no global memory (the next uses, depths and
// masks come four batches at a time through LDS).  A refill syncs at once.
//
// The masks are made for a stretch of accesses at a time, or they would take
// 8.1 bytes per access, many times the bitmaps of a few capacities.  A wave
// leaves its state in memory at a stretch's end and takes it up again in the
// next one's launch.
//
// Bound: the instructions of one wave, batch after batch, at the capacities
// that evict most: 4.0e6 agent accesses at 69 capacities 0.139 s, 2.2 us a
// batch of 64 (0.333 s with the joint ranking of all 128 candidates worked out
// per capacity and a walk per rank and access).
#include "pc_internal.h"

namespace pc {

constexpr uint32_t BEL_TARGET = 96;           // buffer size a refill aims for and a spill leaves
constexpr uint32_t BEL_SPILL_AT = 160;        // buffer size above which the lowest values are spilled
// (a merge moves the whole buffer: 147.5 ms, with 128 and 256 152.2, with 160 and 320 159.3)
// LDS buffer entries: the largest fill (spill size + one batch), and what a
// search reads past a short buffer
constexpr uint32_t BEL_BUF = BEL_SPILL_AT + 3 * WAVE;
constexpr uint64_t BEL_INF = 1ull << 40;      // theta before the first refill: everything in the bitmap
constexpr int32_t DEV_ERR_BELADY = 5;
constexpr uint64_t BEL_RING = 64;             // bitmap words just past the window held in LDS
constexpr uint64_t BEL_SYNC = 16;             // batches between two exchanges with the global bitmap
static_assert(2 * BEL_SYNC <= BEL_RING, "a word entering the ring is merged before the window reaches it");
constexpr int BEL_GROUP = 4;                  // batches whose next[], depth[] and masks are loaded together

__device__ __forceinline__ uint64_t bm_load(const uint64_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t bm_or(uint64_t *p, uint64_t v) {
    return __hip_atomic_fetch_or(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t bm_and(uint64_t *p, uint64_t v) {
    return __hip_atomic_fetch_and(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t bm_xchg(uint64_t *p, uint64_t v) {
    return __hip_atomic_exchange(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// value x into the bitmap: its bit, and its word's bit in the summary
__device__ __forceinline__ void bm_insert(uint64_t *l0, uint64_t *l1, uint32_t x) {
    const uint32_t w = x >> 6;
    bm_or(&l0[w], 1ull << (x & 63));
    bm_or(&l1[w >> 6], 1ull << (w & 63));
}

// every earlier memory operation of the wave completes before later ones
__device__ __forceinline__ void wave_fence() { __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup"); }

__device__ __forceinline__ uint32_t wave_max(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_readlane((int)wave_incl_max(x), WAVE - 1);
}
__device__ __forceinline__ uint64_t wave_or64(uint64_t x) {
    const uint32_t lo = wave_incl_or((uint32_t)x), hi = wave_incl_or((uint32_t)(x >> 32));
    return (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)lo, WAVE - 1) |
           ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)hi, WAVE - 1) << 32);
}
// sum of one uint32 per lane, exact (as two 16-bit halves)
__device__ __forceinline__ uint64_t wave_sum64(uint32_t x) {
    const uint32_t lo = wave_incl_scan(x & 0xFFFFu), hi = wave_incl_scan(x >> 16);
    return (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)lo, WAVE - 1) +
           ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)hi, WAVE - 1) << 16);
}

// next[t] of lane's access (NONE past the end), checked only when used so
// that the load stays in flight until then
__device__ __forceinline__ uint32_t load_next(const uint32_t *__restrict__ next, uint64_t t, uint64_t n) {
    return t < n ? next[t] : NONE;
}
// the loaded next[t], NONE for an invalid entry (flagged)
__device__ __forceinline__ uint32_t checked_next(uint32_t x, uint64_t t, uint64_t n, int32_t *err) {
    if (x != NONE && ((uint64_t)x <= t || (uint64_t)x >= n)) {
        atomicOr(err, DEV_ERR_BAD_LAYOUT);
        return NONE;
    }
    return x;
}

// Number of the descending values buf[0 .. len) above x, from a multiple of
// 64 on that is known to be above x (len at most 512): eight ways at a time,
// three LDS reads in a chain where a binary search has nine.
__device__ __forceinline__ uint32_t above_in(const uint32_t *buf, uint32_t len, uint32_t x, uint32_t from) {
    uint32_t r = 0;
#pragma unroll
    for (uint32_t k = 0; k < 7; ++k) {
        const uint32_t i = from + 8 * k + 7, v = buf[i];
        r += i < len && v > x ? 8u : 0u;
    }
    r += from;
    uint32_t c = 0;
#pragma unroll
    for (uint32_t k = 0; k < 8; ++k) {
        const uint32_t v = buf[r + k];
        c += r + k < len && v > x ? 1u : 0u;
    }
    return r + c;
}
__device__ __forceinline__ uint32_t above_all(const uint32_t *buf, uint32_t len, uint32_t x) {
    uint32_t from = 0;
    for (uint32_t i = WAVE - 1; i < len; i += WAVE) from += buf[i] > x ? (uint32_t)WAVE : 0u;
    // (from = len when all are above)
    return from >= len ? len : above_in(buf, len, x, from);
}

// What a batch's evictions need of next[] alone, once for all capacities, for
// the accesses [from, to): per access the accesses of its batch whose next uses
// lie past the batch and above its own (their number is its rank), and per
// batch the positions that the batch links to inside itself.  One wave per
// batch.
__global__ __launch_bounds__(4 * WAVE) void belady_rank_kernel(const uint32_t *__restrict__ next, uint64_t n,
                                                               uint64_t from, uint64_t to,
                                                               uint64_t *__restrict__ higher,
                                                               uint64_t *__restrict__ links,
                                                               int32_t *__restrict__ err) {
    __shared__ __align__(16) uint32_t s_val[4][WAVE];
    const int lane = threadIdx.x & (WAVE - 1), w = threadIdx.x / WAVE;
    const uint64_t batches = (to - from + WAVE - 1) / WAVE;
    for (uint64_t b0 = (uint64_t)blockIdx.x * 4; b0 < batches; b0 += (uint64_t)gridDim.x * 4) {
        const uint64_t b = b0 + w, at = b * WAVE + lane, t = from + at;
        const uint32_t x = checked_next(load_next(next, t, n), t, n, err);
        const uint64_t we = from + (b + 1) * WAVE;
        const uint32_t v = x != NONE && x >= we ? x : 0u;
        const uint64_t link = wave_or64(x != NONE && x < we ? 1ull << (x & (WAVE - 1)) : 0ull);
        __syncthreads();
        s_val[w][lane] = v;
        __syncthreads();
        const uint4 *q = reinterpret_cast<const uint4 *>(s_val[w]);
        uint32_t m[2] = {0, 0};
#pragma unroll
        for (int i = 0; i < WAVE / 4; ++i) {
            const uint4 a = q[i];
            m[i / 8] |= (uint32_t)(a.x > v) << (4 * i % 32) | (uint32_t)(a.y > v) << (4 * i % 32 + 1) |
                        (uint32_t)(a.z > v) << (4 * i % 32 + 2) | (uint32_t)(a.w > v) << (4 * i % 32 + 3);
        }
        if (t < to) higher[at] = (uint64_t)m[0] | (uint64_t)m[1] << 32;
        if (lane == 0 && b < batches) links[b] = link;
    }
}

// A walk over six accesses: -1 for each bit of v (an eviction), then +1 for
// each bit of i (an insert), access by access; the table holds the lowest sum
// met right after an eviction (none: WALK_NONE, above every sum that counts).
constexpr int WALK = 6, WALK_GROUPS = (WAVE + WALK - 1) / WALK, WALK_NONE = 127;
__device__ __forceinline__ int walk_low(uint32_t v, uint32_t i) {
    int sum = 0, low = WALK_NONE;
    for (int j = 0; j < WALK; ++j) {
        if ((v >> j) & 1) {
            --sum;
            low = sum < low ? sum : low;
        }
        sum += (i >> j) & 1;
    }
    return low;
}

// ---- the simulation of one capacity
struct BelState {
    uint32_t *buf, *alt;   // buf[head .. head + bufn) descending; alt is the spare array
    uint32_t head, bufn;
    uint64_t theta;
    uint64_t bm_hi;        // every bitmap value is below this
    uint64_t *ring;        // LDS: bitmap words [wb, wb + BEL_RING) of window word wb, slot w % BEL_RING
    uint64_t ex_lo;        // ring words from here on may still have bits in the global bitmap
    uint64_t fl_lo;        // ring words [fl_lo, fl_lo + fl_n) were exchanged and are not merged yet:
    uint32_t fl_n;         //   lane i holds word fl_lo + i's bits in fl_val
    uint64_t fl_val;
    uint64_t w0;           // global bitmap words
};

// value x (not in the window) into the bitmap: an LDS ring word when the
// ring holds its word (ring end rend, exclusive, in words), else the global
// bitmap word and its summary bit
__device__ __forceinline__ void bel_insert(const BelState &S, uint64_t *l0, uint64_t *l1, uint32_t x,
                                           uint64_t rend) {
    if ((uint64_t)(x >> 6) < rend)
        atomicOr(reinterpret_cast<unsigned long long *>(&S.ring[(x >> 6) % BEL_RING]), 1ull << (x & 63));
    else
        bm_insert(l0, l1, x);
}

// Brings the ring up to date with the global bitmap for ring end rend: the
// words exchanged at the last sync are merged (their exchanges have returned
// after the fence), and the words that entered the ring since then are taken
// out of the global bitmap (their global inserts are complete after the
// fence).  Those exchanges return during the next batches and are merged at
// the next sync, BEL_SYNC batches before the window can reach them; with
// `full` they are waited for and merged at once.
__device__ __forceinline__ void ring_sync(BelState &S, uint64_t *l0, uint64_t *l1, uint64_t rend, bool full) {
    const int lane = threadIdx.x;
    if (!full && S.fl_n == 0 && S.bm_hi <= (S.ex_lo << 6)) {
        // nothing in flight, and the words to exchange hold no value
        if (rend > S.ex_lo) S.ex_lo = rend;
        return;
    }
    __builtin_amdgcn_s_waitcnt(0);   // this wave's global inserts and exchanges have completed
    wave_fence();
    if ((uint32_t)lane < S.fl_n && S.fl_val)
        atomicOr(reinterpret_cast<unsigned long long *>(&S.ring[(S.fl_lo + lane) % BEL_RING]), S.fl_val);
    const uint64_t m = rend > S.ex_lo ? rend - S.ex_lo : 0;   // at most BEL_SYNC + 1 words
    const uint64_t w = S.ex_lo + lane;
    uint64_t v = 0;
    if ((uint64_t)lane < m && w < S.w0) {
        v = bm_xchg(&l0[w], 0ull);
        bm_and(&l1[w >> 6], ~(1ull << (w & 63)));
    }
    S.fl_lo = S.ex_lo;
    S.fl_n = (uint32_t)m;
    S.fl_val = v;
    if (rend > S.ex_lo) S.ex_lo = rend;
    if (full) {
        __builtin_amdgcn_s_waitcnt(0);
        wave_fence();
        if ((uint32_t)lane < S.fl_n && S.fl_val)
            atomicOr(reinterpret_cast<unsigned long long *>(&S.ring[(S.fl_lo + lane) % BEL_RING]), S.fl_val);
        S.fl_n = 0;
        S.fl_val = 0;
    }
    __syncthreads();
}

// buffer back to index 0 (through the spare array)
__device__ __forceinline__ void compact(BelState &S) {
    if (S.head == 0) return;
    for (uint32_t i = threadIdx.x; i < S.bufn; i += WAVE) S.alt[i] = S.buf[S.head + i];
    __syncthreads();
    uint32_t *tmp = S.buf;
    S.buf = S.alt;
    S.alt = tmp;
    S.head = 0;
}

// the largest bitmap values in [lo, theta) to the buffer's tail until it
// holds BEL_TARGET values: whole words, top down (the global bitmap's words
// past the ring first, the summary skipping empty words, then the ring's);
// theta drops to the lowest value taken.  lo is the window's end and rend
// the ring's end (words).
__device__ void refill(BelState &S, uint64_t *l0, uint64_t *l1, uint64_t lo_all, uint64_t n, uint64_t rend) {
    const int lane = threadIdx.x;
    ring_sync(S, l0, l1, rend, true);   // every ring value in LDS, every insert visible
    compact(S);
    uint64_t hi = S.theta < n + WAVE ? S.theta : n + WAVE;   // exclusive
    if (S.bm_hi < hi) hi = S.bm_hi;
    // global words: values from the ring's end on
    const uint64_t lo = lo_all > (rend << 6) ? lo_all : (rend << 6);
    const uint64_t wlo = lo >> 6;
    const uint64_t lo_mask = ~((1ull << (lo & 63)) - 1);
    while (S.bufn < BEL_TARGET && hi > lo) {
        uint64_t w = (hi - 1) >> 6;
        const uint64_t room = hi - (w << 6);   // 1 .. 64 positions of word w below hi
        uint64_t bits = bm_load(&l0[w]) & (room >= 64 ? ~0ull : (1ull << room) - 1);
        if (w == wlo) bits &= lo_mask;
        if (!bits) {
            // the highest non-empty word below w
            const uint64_t g = w >> 6;
            uint64_t w2 = ~0ull;
            const uint64_t sb = bm_load(&l1[g]) & ((1ull << (w & 63)) - 1);
            if (sb) {
                w2 = (g << 6) + 63 - (uint64_t)__builtin_clzll(sb);
            } else {
                for (int64_t gb = (int64_t)g - 1; gb >= (int64_t)(wlo >> 6); gb -= WAVE) {
                    const int64_t my = gb - lane;
                    const uint64_t v = my >= (int64_t)(wlo >> 6) ? bm_load(&l1[my]) : 0ull;
                    const uint64_t nz = ballot(v != 0);
                    if (nz) {
                        const int L = __builtin_ctzll(nz);
                        const uint64_t vv = readlane64(v, L);
                        w2 = ((uint64_t)(gb - L) << 6) + 63 - (uint64_t)__builtin_clzll(vv);
                        break;
                    }
                }
            }
            if (w2 == ~0ull || w2 < wlo) {   // nothing left in [lo, hi)
                hi = lo;
                break;
            }
            w = w2;
            bits = bm_load(&l0[w]);
            if (w == wlo) bits &= lo_mask;
            if (!bits) {   // a stale summary bit: go on below this word
                hi = w << 6 > lo ? w << 6 : lo;
                continue;
            }
        }
        // the word's values, largest first
        if ((bits >> lane) & 1) {
            const uint64_t above = lane == WAVE - 1 ? 0ull : bits & (~0ull << (lane + 1));
            S.buf[S.bufn + (uint32_t)__popcll(above)] = (uint32_t)((w << 6) + lane);
        }
        S.bufn += (uint32_t)__popcll(bits);
        const uint64_t low = (w << 6) + (uint64_t)__builtin_ctzll(bits);
        S.theta = low;
        if (lane == 0) {
            const uint64_t old = bm_and(&l0[w], ~bits);
            if ((old & ~bits) == 0) bm_and(&l1[w >> 6], ~(1ull << (w & 63)));
        }
        hi = w << 6 > lo ? w << 6 : lo;
    }
    // ring words, top down, when the global ones did not suffice
    if (hi > lo_all && hi <= lo) {
        const uint64_t rlo_mask = ~((1ull << (lo_all & 63)) - 1);
        while (S.bufn < BEL_TARGET && hi > lo_all) {
            const uint64_t w = (hi - 1) >> 6;
            const uint64_t room = hi - (w << 6);
            uint64_t bits = S.ring[w % BEL_RING] & (room >= 64 ? ~0ull : (1ull << room) - 1);
            if (w == (lo_all >> 6)) bits &= rlo_mask;
            if (bits) {
                if ((bits >> lane) & 1) {
                    const uint64_t above = lane == WAVE - 1 ? 0ull : bits & (~0ull << (lane + 1));
                    S.buf[S.bufn + (uint32_t)__popcll(above)] = (uint32_t)((w << 6) + lane);
                }
                S.bufn += (uint32_t)__popcll(bits);
                S.theta = (w << 6) + (uint64_t)__builtin_ctzll(bits);
                __syncthreads();
                if (lane == 0) S.ring[w % BEL_RING] &= ~bits;
                __syncthreads();
            }
            hi = w << 6 > lo_all ? w << 6 : lo_all;
        }
    }
    // every bitmap value at or above hi has been taken
    if (hi < S.bm_hi) S.bm_hi = hi > lo_all ? hi : lo_all;
    __syncthreads();
}

// the buffer's top 64 values, one per lane (0 past its end)
__device__ __forceinline__ uint32_t buffer_top(const BelState &S) {
    return (uint32_t)threadIdx.x < S.bufn ? S.buf[S.head + threadIdx.x] : 0u;
}

__device__ __forceinline__ uint32_t clamp32(uint64_t v) { return v > 0xFFFFFFFFull ? 0xFFFFFFFFu : (uint32_t)v; }

// four words at any 4-byte alignment
struct __attribute__((packed, aligned(4))) BelQuad {
    uint32_t x, y, z, w;
};
struct BelGroup {
    alignas(16) uint32_t next[BEL_GROUP][WAVE], depth[BEL_GROUP][WAVE];
    static_assert(BEL_GROUP == 4, "a lane loads four accesses of a group");
    alignas(16) uint64_t higher[BEL_GROUP][WAVE];
    uint64_t link[BEL_GROUP];
};

// What a capacity's wave hands from one stretch to the next.
struct BelSaved {
    uint64_t ring[BEL_RING], fl_val[WAVE];
    uint64_t theta, bm_hi, ex_lo, fl_lo, hits, dsum;
    uint32_t buf[BEL_BUF];
    uint32_t bufn, fl_n, dead, size;
    uint32_t stopped;   // 0 once the stretch is through: if a check ended it, the later ones do nothing
};

// The accesses [from, to), `from` a multiple of BEL_STRETCH: 0, or the state
// is resumed.  `higher` and `links` are indexed as if they held all accesses;
// saved: nullptr when there is one stretch only.  The loop is short of scalar
// registers, so nothing is added to it that can wait elsewhere.
template <bool RESUME>
__device__ void belady_one(const uint32_t *__restrict__ next, const uint32_t *__restrict__ depth, uint64_t n,
                           uint64_t from, uint64_t to, BelSaved *saved,
                           uint64_t c64, uint64_t *__restrict__ l0, uint64_t *__restrict__ l1, uint64_t w0,
                           const uint64_t *__restrict__ higher, const uint64_t *__restrict__ links,
                           uint8_t *__restrict__ flags, uint64_t *hits_out, uint64_t *dsum_out, int32_t *err,
                           uint32_t *s_a, uint32_t *s_b, uint32_t *s_new, uint8_t *s_mark, const int8_t *s_walk,
                           uint64_t *s_ring, BelGroup &L) {
    const int lane = threadIdx.x;
    // the global bitmap starts empty, so the ring's first words are complete
    BelState S{s_a, s_b, 0, 0, BEL_INF, 0, s_ring, BEL_RING, 0, 0, 0, w0};
    for (uint64_t i = lane; i < BEL_RING; i += WAVE) s_ring[i] = 0;
    // (next[] that is not one-to-one leaves places of the buffer unwritten)
    for (uint32_t i = lane; i < BEL_BUF; i += WAVE) s_a[i] = s_b[i] = 0;
    s_new[lane] = 0;
    __syncthreads();
    // resident blocks never exceed n, so the capacity is clamped to 32 bits
    const uint32_t c = clamp32(c64 < n ? c64 : n);
    uint32_t dead = 0, size = 0;
    uint64_t hits = 0, dsum = 0;
    if constexpr (RESUME) {
        if (saved->stopped) return;
        S.bufn = (uint32_t)__builtin_amdgcn_readfirstlane((int)saved->bufn);
        S.theta = readlane64(saved->theta, 0);
        S.bm_hi = readlane64(saved->bm_hi, 0);
        S.ex_lo = readlane64(saved->ex_lo, 0);
        S.fl_lo = readlane64(saved->fl_lo, 0);
        S.fl_n = (uint32_t)__builtin_amdgcn_readfirstlane((int)saved->fl_n);
        S.fl_val = saved->fl_val[lane];
        dead = (uint32_t)__builtin_amdgcn_readfirstlane((int)saved->dead);
        size = (uint32_t)__builtin_amdgcn_readfirstlane((int)saved->size);
        hits = readlane64(saved->hits, 0);
        dsum = readlane64(saved->dsum, 0);
        for (uint64_t i = lane; i < BEL_RING; i += WAVE) s_ring[i] = saved->ring[i];
        for (uint32_t i = lane; i < S.bufn; i += WAVE) s_a[i] = saved->buf[i];
        __syncthreads();
    }
    // (a wave that an internal check stops leaves the mark)
    if (saved && lane == 0) saved->stopped = 1;
    // what only the end needs waits in LDS
    __shared__ BelSaved *s_saved;
    __shared__ uint64_t *s_out[2];
    s_saved = saved;
    s_out[0] = hits_out;
    s_out[1] = dsum_out;
    uint32_t n32 = (uint32_t)n;   // (in a vector register)
    __asm__ volatile("" : "+v"(n32));
    auto length = [&]() { return (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)n32); };
    const int own = lane / WALK, own_at = own * WALK;   // the lane's group of the walk, its first access
    // A group's next uses, depths and masks lie in LDS, and the next group's
    // are on their way in registers: a batch that waited for a load of its own
    // would wait for the newest one too, and for its inserts into the bitmap.
    const uint64_t batches = (to + WAVE - 1) / WAVE;
    // each lane four consecutive accesses, one load per array
    BelQuad xa, da{0, 0, 0, 0}, ha0, ha1;
    uint64_t lk = 0;   // the links of the group's batches, one per lane
    auto load_group = [&](uint64_t b0) {
        const uint64_t t = b0 * WAVE + 4 * lane;
        if ((b0 + BEL_GROUP) * WAVE <= to) {
            xa = *reinterpret_cast<const BelQuad *>(next + t);
            if (depth) da = *reinterpret_cast<const BelQuad *>(depth + t);
            ha0 = reinterpret_cast<const BelQuad *>(higher + t)[0];
            ha1 = reinterpret_cast<const BelQuad *>(higher + t)[1];
        } else {
            auto one = [&](const uint32_t *p, uint64_t k, uint64_t m, uint32_t none) { return k < m ? p[k] : none; };
            xa = BelQuad{one(next, t, to, NONE), one(next, t + 1, to, NONE), one(next, t + 2, to, NONE),
                         one(next, t + 3, to, NONE)};
            if (depth) da = BelQuad{one(depth, t, to, 0), one(depth, t + 1, to, 0), one(depth, t + 2, to, 0),
                                    one(depth, t + 3, to, 0)};
            const uint32_t *h = reinterpret_cast<const uint32_t *>(higher);
            const uint64_t u = 2 * t, m = 2 * to;
            ha0 = BelQuad{one(h, u, m, 0), one(h, u + 1, m, 0), one(h, u + 2, m, 0),
                          one(h, u + 3, m, 0)};
            ha1 = BelQuad{one(h, u + 4, m, 0), one(h, u + 5, m, 0), one(h, u + 6, m, 0),
                          one(h, u + 7, m, 0)};
        }
        if (lane < BEL_GROUP) lk = b0 + lane < batches ? links[b0 + lane] : 0ull;
    };
    load_group(from / WAVE);
    for (uint64_t t0 = from; t0 < to; t0 += WAVE) {
        const int in_group = (int)((t0 / WAVE) % BEL_GROUP);
        if (in_group == 0) {
            __syncthreads();
            const uint64_t t = t0 + 4 * lane;
            reinterpret_cast<uint4 *>(L.next)[lane] =
                make_uint4(checked_next(xa.x, t, n32, err), checked_next(xa.y, t + 1, n32, err),
                           checked_next(xa.z, t + 2, n32, err), checked_next(xa.w, t + 3, n32, err));
            reinterpret_cast<uint4 *>(L.depth)[lane] = make_uint4(da.x, da.y, da.z, da.w);
            reinterpret_cast<uint4 *>(L.higher)[2 * lane] = make_uint4(ha0.x, ha0.y, ha0.z, ha0.w);
            reinterpret_cast<uint4 *>(L.higher)[2 * lane + 1] = make_uint4(ha1.x, ha1.y, ha1.z, ha1.w);
            if (lane < BEL_GROUP) L.link[lane] = lk;
            __syncthreads();
            load_group(t0 / WAVE + BEL_GROUP);
        }
        const uint32_t xq = L.next[in_group][lane], dq = L.depth[in_group][lane];
        const uint64_t hi_mask = L.higher[in_group][lane];
        const uint32_t rank = (uint32_t)__popcll(hi_mask);
        const uint64_t t = t0 + lane;
        const bool valid = t < to;
        const uint32_t xv = xq, dv = dq;
        const int nb = to - t0 < (uint64_t)WAVE ? (int)(to - t0) : WAVE;
        const uint64_t vmask = nb == WAVE ? ~0ull : (1ull << nb) - 1;
        const uint64_t we = t0 + WAVE;
        const uint32_t we32 = clamp32(we), t32 = (uint32_t)t0;

        // keep the buffer out of this batch's positions: its values inside the
        // window join the window word.  They are its smallest ones (the buffer
        // is descending and holds no value below the window), distinct
        // positions of the window, so at most its last 64 entries, one per lane.
        uint64_t wlow = 0;
        if (S.theta < we) {
            const uint32_t bn = S.bufn;
            const bool has = (uint32_t)lane < bn;
            const uint32_t v = has ? S.buf[S.head + bn - 1 - lane] : NONE;
            const bool in = has && (uint64_t)v < we;
            wlow = wave_or64(in ? 1ull << (v - t32) : 0ull);
            S.bufn = bn - (uint32_t)__popcll(ballot(in));
            S.theta = we;
        }

        // values present in the window: that register and the window's ring
        // word (complete: merged at a sync at least BEL_SYNC batches ago),
        // taken and cleared; the ring now ends BEL_RING words past the window
        const uint64_t w = t0 >> 6;
        const uint64_t rend = w + BEL_RING;
        uint64_t wbits = wlow;
        if (S.bm_hi > t0) {   // else the bitmap holds nothing at or past the window
            wbits |= S.ring[w % BEL_RING];
            __syncthreads();
            if (lane == 0) S.ring[w % BEL_RING] = 0;
            __syncthreads();
        }
        const uint64_t link = readlane64(L.link[in_group], 0);   // (uniform)
        uint64_t hm = (wbits | link) & vmask;
        const uint32_t misses = (uint32_t)__popcll(vmask & ~hm);
        const uint32_t E = size + misses > c ? size + misses - c : 0u;
        if (E > dead && dead + S.bufn < (uint32_t)WAVE) refill(S, l0, l1, we, length(), rend);

        bool to_buffer, to_bitmap;
        uint32_t popped = 0;
        uint32_t above = NONE;   // buffer values above this lane's (before any is popped), once known
        uint32_t order = rank;   // rank among the values that go to the buffer
        if (E <= dead) {
            // nothing in the window can leave: bulk
            dead += (uint32_t)__popcll(ballot(valid && xv == NONE)) - E;
            size = size + misses - E;
            to_buffer = valid && xv != NONE && xv >= we32 && (uint64_t)xv >= S.theta;
            to_bitmap = valid && xv != NONE && xv >= we32 && (uint64_t)xv < S.theta;
        } else {
            // The candidates: the batch's inserts above the window (pending) and
            // the buffer's top 64 values, ranked jointly.
            const bool pend = valid && xv != NONE && xv >= we32;
            const uint64_t pmask = ballot(pend);
            const uint32_t np = (uint32_t)__popcll(pmask);
            const uint32_t nbt = S.bufn < (uint32_t)WAVE ? S.bufn : (uint32_t)WAVE;
            const uint32_t in_top = above_in(S.buf + S.head, nbt, xv, 0);   // of those, the ones above this lane's
            if (in_top < nbt || nbt == S.bufn) above = in_top;
            // below theta the bitmap may hold larger values, which only the
            // general walk below handles
            const uint64_t high = ballot(pend && (uint64_t)xv >= S.theta);
            // evictions: the misses after the cache has filled up
            uint64_t ev = vmask & ~hm;
            for (uint32_t k = size; k < c && ev; ++k) ev &= ev - 1;
            const uint64_t dm = ballot(valid && xv == NONE);
            // (1) Evictions that find no dead block.  With D(j) evictions up to
            // and including access j and S(j) dead blocks available before it
            // (a dead insert counts from the next access on), the number left
            // unserved is the running maximum of D(j) - S(j): the real
            // evictions are the accesses where that maximum grows.
            const uint64_t le = lane == WAVE - 1 ? ~0ull : (2ull << lane) - 1;   // lanes up to this one
            const int64_t gap = (int64_t)__popcll(ev & le) - (int64_t)dead - (int64_t)__popcll(dm & (le >> 1));
            const uint32_t un = wave_incl_max(gap > 0 ? (uint32_t)gap : 0u);
            // (wave_shr:1, 0 into lane 0)
            const uint32_t un_prev = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)un, 0x138, 0xf, 0xf, false);
            const uint64_t real = ballot(un > un_prev);
            const uint32_t n_real = (uint32_t)__popcll(real);
            // (2) Which candidates the real evictions take.  Each takes the
            // largest one present; the buffer's are present from the start, a
            // pending one after its own access.  For a value x let R(x) be the
            // number of evictions that take a candidate above x.  With A(x)
            // buffer candidates above x, and r_i the count after the i-th
            // eviction, r_i = min(r_{i-1} + 1, A(x) + P_i(x)) where P_i(x)
            // counts the pending candidates above x inserted before it, hence
            // R(x) = min(n, A(x) + n + m(x)) with n of them in all (n_real) and m(x)
            // the lowest sum of the walk "-1 per eviction, then +1 per such insert",
            // access by access.
            // x itself is taken iff counting it too makes R larger: iff the walk
            // gets, after x's own access, below both -A(x) and every sum before.
            // Each lane walks for its own value, six accesses per table entry.
            // (Below every sum before its own access, and -A(x): then the lowest of
            // all is also the lowest after it.)
            int in = 0, all = 0, pre = -(int)in_top;
            int8_t low[WALK_GROUPS];
#pragma unroll
            for (int g = 0; g < WALK_GROUPS; ++g)
                low[g] = s_walk[((uint32_t)(real >> (WALK * g)) & 63) * 64 + ((uint32_t)(hi_mask >> (WALK * g)) & 63)];
            const uint64_t before = (1ull << own_at) - 1;   // the groups before the lane's own
            const uint32_t upto = (2u << (lane - own_at)) - 1;
            const int own_pre = s_walk[((uint32_t)(real >> own_at) & 63 & upto) * 64 +
                                       ((uint32_t)(hi_mask >> own_at) & 63)] +
                                (int)__popcll(hi_mask & before) - (int)__popcll(real & before);
#pragma unroll
            for (int g = 0; g < WALK_GROUPS; ++g) {
                const int x = in - (int)__popcll(real & ((1ull << (WALK * g)) - 1)) + (int)low[g];
                all = x < all ? x : all;
                const int y = g < own ? x : 0;
                pre = y < pre ? y : pre;
                in += (int)__popc((uint32_t)(hi_mask >> (WALK * g)) & 63);
            }
            pre = own_pre < pre ? own_pre : pre;
            const uint64_t gone_if = ballot(pend && all < pre);
            // all real evictions find a candidate at or above theta
            const uint64_t lt = (1ull << lane) - 1;
            const int sum = (int)__popcll(high & lt) - (int)__popcll(real & le);
            const bool ok = ballot(((real >> lane) & 1) && sum < -(int)nbt) == 0;
            const uint32_t d = dead + (uint32_t)__popcll(dm) - ((uint32_t)__popcll(ev) - n_real);
            uint64_t gone = 0;   // lane mask
            if (ok) {
                dead = d;
                size = c;   // evictions happened, so the cache is full
                gone = gone_if;
                popped = n_real - (uint32_t)__popcll(gone);
                // With next[] one-to-one the buffer gives the rest of the
                // evictions; copies of a value each count as taken, so that
                // more may be gone than were evicted.
                if (popped > S.bufn) {   // (below 0 too: the count wraps)
                    if (lane == 0) atomicOr(err, DEV_ERR_BELADY);
                    return;
                }
            } else {
            // the general walk: the window in a register, a refill when the
            // buffer and the batch's inserts above theta run out, the window's
            // largest value when nothing above the window is left
            __syncthreads();
            if (pend) s_new[rank] = xv;
            __syncthreads();
            const uint32_t sorted = (uint32_t)lane < np ? s_new[lane] : 0u;
            uint32_t top = buffer_top(S);
            uint64_t avail = 0, rgone = 0;   // by pending rank: inserted so far / evicted again
            uint64_t wreg = wbits;
            hm = 0;
            for (int j = 0; j < nb; ++j) {
                const uint64_t bit = 1ull << j;
                const uint32_t x = (uint32_t)__builtin_amdgcn_readlane((int)xv, j);
                if (wreg & bit) {
                    wreg &= ~bit;
                    hm |= bit;
                } else if (size < c) {
                    ++size;
                } else if (dead) {
                    --dead;
                } else {
                    const uint64_t cand = avail & ~rgone;   // lowest rank = largest value
                    const uint32_t pm = cand ? (uint32_t)__builtin_amdgcn_readlane((int)sorted, __builtin_ctzll(cand)) : 0u;
                    uint32_t pb = popped < S.bufn ? (uint32_t)__builtin_amdgcn_readlane((int)top, popped) : 0u;
                    if (pb == 0 && pm < clamp32(S.theta)) {
                        // buffer exhausted and the bitmap may hold larger values
                        S.head += popped;
                        S.bufn -= popped;
                        popped = 0;
                        above = NONE;
                        refill(S, l0, l1, we, length(), rend);
                        top = buffer_top(S);
                        pb = S.bufn ? (uint32_t)__builtin_amdgcn_readlane((int)top, 0) : 0u;
                    }
                    if (pm > pb) {
                        rgone |= cand & (~cand + 1);
                    } else if (pb) {
                        ++popped;
                    } else if (wreg & ~((bit << 1) - 1)) {
                        // nothing resident above the window: its largest value
                        wreg &= ~(1ull << (63 - __builtin_clzll(wreg)));
                    } else {   // nothing to evict: cannot happen with c resident blocks
                        if (lane == 0) atomicOr(err, DEV_ERR_BELADY);
                        return;
                    }
                }
                // lane j's block stays resident with its next use
                if (x == NONE) {
                    ++dead;
                } else if (x < we32) {
                    wreg |= 1ull << (x - t32);
                } else {
                    avail |= 1ull << (uint32_t)__builtin_amdgcn_readlane((int)rank, j);
                }
            }
            gone = ballot(pend && ((rgone >> rank) & 1));
            }
            const bool alive = pend && !((gone >> lane) & 1);
            to_buffer = alive && (uint64_t)xv >= S.theta;
            to_bitmap = alive && (uint64_t)xv < S.theta;
            order = rank - (uint32_t)__popcll(hi_mask & gone);
        }

        // the batch's results
        const bool h = (hm >> lane) & 1;
        hits += (uint64_t)__popcll(hm);
        dsum += wave_sum64(h ? dv : 0u);
        if (flags && valid) flags[t] = h ? 1 : 0;
        if (ballot(to_bitmap)) {
            if (to_bitmap) bel_insert(S, l0, l1, xv, rend);
            const uint64_t m = (uint64_t)wave_max(to_bitmap ? xv : 0u) + 1;
            if (m > S.bm_hi) S.bm_hi = m;
        }

        // buffer: drop the popped values, merge the batch's values above theta
        S.head += popped;
        S.bufn -= popped;
        const uint64_t alive = ballot(to_buffer);
        const uint32_t nn = (uint32_t)__popcll(alive);
        if (nn) {
            // (values go to the buffer from the largest on, so `order` counts
            // from 0 without gaps); buffer values above it, after the popped ones
            uint32_t lo;
            if (ballot(to_buffer && above == NONE)) {
                lo = above_all(S.buf + S.head, S.bufn, xv);
            } else {
                lo = above > popped ? above - popped : 0u;
            }
            // marks at the new values' places; the others keep their order
            __syncthreads();
            reinterpret_cast<uint64_t *>(s_mark)[lane] = 0;
            __syncthreads();
            if (to_buffer) {
                s_new[order] = xv;
                s_mark[order + lo] = 1;
            }
            __syncthreads();
            const uint32_t len = S.bufn + nn;
            uint32_t before = 0;   // new values ahead of the chunk
            for (uint32_t p0 = 0; p0 < len; p0 += WAVE) {
                const uint32_t p = p0 + lane;
                const bool is_new = s_mark[p] != 0;
                const uint64_t m = ballot(is_new);
                const uint32_t k = before + mbcnt(m);
                if (p < len) S.alt[p] = is_new ? s_new[k] : S.buf[S.head + p - k];
                before += (uint32_t)__popcll(m);
            }
            __syncthreads();
            uint32_t *tmp = S.buf;
            S.buf = S.alt;
            S.alt = tmp;
            S.head = 0;
            S.bufn += nn;
        }
        // spill the lowest values when the buffer grows large
        if (S.bufn > BEL_SPILL_AT) {
            const uint64_t top_spilled = (uint64_t)S.buf[S.head + BEL_TARGET] + 1;
            for (uint32_t i = BEL_TARGET + lane; i < S.bufn; i += WAVE)
                bel_insert(S, l0, l1, S.buf[S.head + i], rend);
            if (top_spilled > S.bm_hi) S.bm_hi = top_spilled;
            S.bufn = BEL_TARGET;
            S.theta = S.buf[S.head + BEL_TARGET - 1];
        }
        __syncthreads();
        // every BEL_SYNC batches: the ring against the global bitmap, for the
        // next batch's ring end
        if ((w + 1) % BEL_SYNC == 0) ring_sync(S, l0, l1, rend + 1, false);
    }
    if (to < length()) {
        saved = s_saved;
        for (uint64_t i = lane; i < BEL_RING; i += WAVE) saved->ring[i] = s_ring[i];
        for (uint32_t i = lane; i < S.bufn; i += WAVE) saved->buf[i] = S.buf[S.head + i];
        saved->fl_val[lane] = S.fl_val;
        if (lane == 0) {
            saved->bufn = S.bufn;
            saved->theta = S.theta;
            saved->bm_hi = S.bm_hi;
            saved->ex_lo = S.ex_lo;
            saved->fl_lo = S.fl_lo;
            saved->fl_n = S.fl_n;
            saved->dead = dead;
            saved->size = size;
            saved->hits = hits;
            saved->dsum = dsum;
            saved->stopped = 0;
        }
        return;
    }
    if (lane == 0) {
        *s_out[0] = hits;
        *s_out[1] = dsum;
    }
}

template <bool RESUME>
__global__ __launch_bounds__(WAVE) void belady_kernel(const uint32_t *__restrict__ next,
                                                      const uint32_t *__restrict__ depth, uint64_t n,
                                                      uint64_t from, uint64_t to, BelSaved *__restrict__ saved,
                                                      const uint64_t *__restrict__ caps, uint64_t *__restrict__ l0s,
                                                      uint64_t *__restrict__ l1s, uint64_t w0, uint64_t w1,
                                                      const uint64_t *__restrict__ higher,
                                                      const uint64_t *__restrict__ links,
                                                      uint64_t *__restrict__ hits, uint64_t *__restrict__ dsum,
                                                      uint8_t *__restrict__ flags, int32_t *__restrict__ err) {
    __shared__ uint32_t s_a[BEL_BUF], s_b[BEL_BUF], s_new[WAVE];
    __shared__ __align__(8) uint8_t s_mark[8 * WAVE];
    __shared__ int8_t s_walk[64 * 64];
    __shared__ BelGroup s_group;
    for (int i = threadIdx.x; i < 64 * 64; i += WAVE) s_walk[i] = (int8_t)walk_low((uint32_t)i / 64, (uint32_t)i % 64);
    __syncthreads();
    __shared__ uint64_t s_ring[BEL_RING];
    const uint32_t k = blockIdx.x;
    const uint64_t c = caps[k];
    uint8_t *fl = flags ? flags + (uint64_t)k * n : nullptr;
    if (c == 0) {
        if (from > 0) return;
        if (fl)
            for (uint64_t t = threadIdx.x; t < n; t += WAVE) fl[t] = 0;
        if (threadIdx.x == 0) {
            hits[k] = 0;
            dsum[k] = 0;
        }
        return;
    }
    belady_one<RESUME>(next, depth, n, RESUME ? from : 0, to, saved ? saved + k : nullptr, c, l0s + (uint64_t)k * w0,
                       l1s + (uint64_t)k * w1, w0, higher, links, fl, hits + k, dsum + k, err, s_a, s_b, s_new,
                       s_mark, s_walk, s_ring, s_group);
}

// bitmap words per capacity: one bit per position plus a word of slack, and
// the summary (one bit per bitmap word)
static uint64_t bel_w0(uint64_t n) { return (n + 2 * WAVE) / 64 + 1; }
static uint64_t bel_w1(uint64_t n) { return bel_w0(n) / 64 + 2; }

// Accesses per stretch: 136 MB of masks.  At its end all capacities wait for the
// slowest: 2.8e7 accesses at 69 capacities 979 ms, in one stretch 973, in
// stretches of 2^22 992.
constexpr uint64_t BEL_STRETCH = 1ull << 24;
static_assert(BEL_STRETCH % (BEL_GROUP * WAVE) == 0 && BEL_STRETCH % (BEL_SYNC * WAVE) == 0, "stretches are whole groups");
struct BelWs {
    int32_t *hdr;
    uint64_t *l0, *l1, *links, *higher;
    BelSaved *saved;
    size_t bytes;
};
static BelWs bel_ws(void *ws, uint64_t n, uint32_t n_caps) {
    Carver c{(char *)ws, 0};
    BelWs w;
    w.hdr = c.take<int32_t>(WS_HEADER / sizeof(int32_t));
    w.l0 = c.take<uint64_t>(n_caps * (bel_w0(n) + bel_w1(n)));
    w.l1 = w.l0 + n_caps * bel_w0(n);
    const uint64_t m = n < BEL_STRETCH ? n : BEL_STRETCH;
    w.links = c.take<uint64_t>((m + WAVE - 1) / WAVE);
    w.higher = c.take<uint64_t>(m);
    w.saved = n > BEL_STRETCH ? c.take<BelSaved>(n_caps) : nullptr;
    w.bytes = c.off;
    return w;
}

}  // namespace pc

extern "C" {

size_t pc_belady_ws(uint64_t n, uint32_t n_caps) { return pc::bel_ws(nullptr, n, n_caps).bytes; }

pc_status pc_belady(const uint32_t *next, const uint32_t *depth, uint64_t n, const uint64_t *caps, uint32_t n_caps,
                    uint64_t *hits, uint64_t *depthsum, uint8_t *hit_flags, void *ws, size_t ws_bytes,
                    void *stream) {
    if (n >= (uint64_t)PC_NONE) return PC_ERR_TOO_LARGE;
    if (n_caps == 0 || n_caps > PC_MAX_CAPS) return PC_ERR_INVALID;
    if (!caps || !hits || !depthsum) return PC_ERR_INVALID;
    if (n > 0 && !next) return PC_ERR_INVALID;
    if (!ws) return PC_ERR_WORKSPACE;
    if (ws_bytes < pc_belady_ws(n, n_caps)) return PC_ERR_WORKSPACE;
    hipStream_t s = (hipStream_t)stream;
    const pc::BelWs w = pc::bel_ws(ws, n, n_caps);
    const uint64_t w0 = pc::bel_w0(n), w1 = pc::bel_w1(n);
    pc::Fills f;
    f.add(w.hdr, 0u, 1);
    f.add(w.l0, 0u, 2 * (size_t)n_caps * (w0 + w1));
    const pc_status st = pc::fill_all(f, s);
    if (st != PC_OK) return st;
    uint64_t from = 0;
    do {
        const uint64_t to = n - from < pc::BEL_STRETCH ? n : from + pc::BEL_STRETCH;
        if (to > from) {
            const uint64_t per = 4 * pc::WAVE, groups = (to - from + per - 1) / per;
            const uint64_t most = (uint64_t)pc::device_cus() * 16;
            PC_LAUNCH(pc::K_BELADY_RANK, pc::belady_rank_kernel, dim3((unsigned)(groups < most ? groups : most)),
                      dim3(4 * pc::WAVE), 0, s, next, n, from, to, w.higher, w.links, w.hdr);
        }
        const auto kernel = from ? pc::belady_kernel<true> : pc::belady_kernel<false>;
        PC_LAUNCH(pc::K_BELADY, kernel, dim3(n_caps), dim3(pc::WAVE), 0, s, next, depth, n, from, to, w.saved, caps,
                  w.l0, w.l1, w0, w1, w.higher - from, w.links - from / pc::WAVE, hits, depthsum, hit_flags, w.hdr);
        from = to;
    } while (from < n);
    return PC_OK;
}

}  // extern "C"
