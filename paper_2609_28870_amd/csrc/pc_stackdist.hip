// Exact LRU stack distance (pc_stack_distance).
//
// Definition: D(t) = #{ i in (prev(t), t) : next(i) > t }, the number of
// distinct blocks touched since the previous use; an LRU cache of c blocks
// hits exactly when D < c (LRU is a stack algorithm; Sec. 5 "LRU as a
// bedrock", Appendix B "stack distance between reuses").
//
// Reformulation used here.  With v(j) = prev(j) + 1 (0 for a cold access),
// the number of j < t with v(j) < v(t) is prev(t) + 1 + D(t): every i <=
// prev(t) qualifies, and in the window (prev(t), t) exactly the first use of
// each distinct block does.  Non-cold v are distinct, so with Z(t) = number of
// cold accesses before t and C'(t) = #{ non-cold j < t : v(j) < v(t) }:
//        D(t) = Z(t) + C'(t) - v(t).
// C' is a two-dimensional dominance count.  The non-cold accesses are taken in
// v order -- that is just next[] read in index order, since next[p] = t
// exactly when v(t) = p + 1 -- and partitioned by the bits of t from the top
// (MSD radix).  At every level an element adds the number of elements that
// precede it in v order, sit in the same bucket (same higher bits of t) and
// carry a smaller digit.  Summed over all levels this is exactly C'(t), and
// the last level leaves every element at its own t.
//
// Buckets are ranges of t, so their sizes are known in advance from the
// per-4096 prefix of cold counts: #non-cold t < X = X - Z(X).
//   * sd_cold_count + a two-step scan -> Z at every multiple of 4096
//   * per level (1-3 levels of 8-bit digits above bit 12), over tiles of 2048
//     elements: sd_count (per-tile digit counts), a segmented scan of those
//     counts over the tiles of each bucket (sd_seg: reduce, carry, scan --
//     no waiting on other workgroups), then sd_dominance_pass: one ballot
//     per digit bit gives every lane the earlier lanes of its 64-lane chunk
//     with a smaller / equal digit, a 2-D prefix over
//     (chunk, digit) in LDS extends that to the tile, the scanned counts
//     extend it across tiles, and the tile is written out digit-partitioned
//     through LDS.
//   * sd_local_finish -> one workgroup per 4096-range of t: two in-LDS levels
//     of 6 bits finish the count, then D is written in t order with the cold
//     prefix from a block scan.
#include "pc_internal.h"

namespace pc {

constexpr int LOCAL_BITS = 12;
constexpr uint32_t LOCAL_SPAN = 1u << LOCAL_BITS;   // 4096
constexpr int DOM_THREADS = 512;
constexpr int DOM_WAVES = DOM_THREADS / WAVE;
constexpr int DOM_CHUNKS_PER_WAVE = 4;
constexpr int DOM_CHUNKS = DOM_WAVES * DOM_CHUNKS_PER_WAVE;   // 32
constexpr int DOM_TILE = DOM_CHUNKS * WAVE;                    // 2048
constexpr int DOM_RADIX = 256;
static_assert(DOM_THREADS == 2 * DOM_RADIX, "the column prefix splits the chunks in two halves");
constexpr int LOC_THREADS = 512;
constexpr int LOC_WAVES = LOC_THREADS / WAVE;
constexpr int LOC_CHUNKS = LOCAL_SPAN / WAVE;                  // 64
constexpr int LOC_CPW = LOC_CHUNKS / LOC_WAVES;                // 8
constexpr int LOC_PARTS = LOC_THREADS / 64;                    // column-prefix parts per digit
constexpr int SCAN_THREADS = 1024;

// number of non-cold accesses t < X (X a multiple of 4096, or X = n)
__device__ __forceinline__ uint64_t cnt_lt(uint64_t X, const uint32_t *Zc) {
    return X - Zc[(X + LOCAL_SPAN - 1) >> LOCAL_BITS];
}

// The steps below are functions of one chunk of their work, so that the
// kernels (one launch per step) and the persistent kernel (all of them in one
// launch, for callers that seldom need them) share them.

// cold accesses of one 4096-range of t
template <int THREADS>
__device__ __forceinline__ void cold_count(const uint32_t *prev, uint64_t n, uint64_t chunk, uint32_t *cnt,
                                           uint32_t *tmp) {
    // 16-byte vectors, all in flight at once
    constexpr int PER = LOCAL_SPAN / 4 / THREADS;
    const uint64_t base = chunk * LOCAL_SPAN;
    uint32_t c = 0;
    if (base + LOCAL_SPAN <= n && (reinterpret_cast<uintptr_t>(prev) & 15) == 0) {
        const uint4 *p = reinterpret_cast<const uint4 *>(prev + base);
        uint4 v[PER];
#pragma unroll
        for (int q = 0; q < PER; ++q) v[q] = p[threadIdx.x + q * THREADS];
#pragma unroll
        for (int q = 0; q < PER; ++q)
            c += (v[q].x == NONE) + (v[q].y == NONE) + (v[q].z == NONE) + (v[q].w == NONE);
    } else {
        for (uint32_t j = threadIdx.x; j < LOCAL_SPAN; j += THREADS)
            c += (base + j < n && prev[base + j] == NONE) ? 1u : 0u;
    }
    uint32_t total;
    block_excl_scan(c, tmp, &total);
    if (threadIdx.x == 0) cnt[chunk] = total;
}

// Exclusive scan of m values, SCAN_BLOCK per workgroup: block sums first (not
// needed for a single block), then every block adds the sums before its own.
// out[m] = total.
constexpr int SCAN_BLOCK = 4096;
__device__ __forceinline__ void scan_reduce(const uint32_t *in, uint64_t m, uint64_t block, uint32_t *part,
                                            uint32_t *tmp) {
    uint32_t x = 0;
    for (uint32_t j = threadIdx.x; j < SCAN_BLOCK; j += blockDim.x) {
        const uint64_t i = block * SCAN_BLOCK + j;
        x += i < m ? in[i] : 0u;
    }
    uint32_t total;
    block_excl_scan(x, tmp, &total);
    if (threadIdx.x == 0) part[block] = total;
}
template <int THREADS>
__device__ __forceinline__ void scan_apply(const uint32_t *in, uint64_t m, uint64_t block, const uint32_t *part,
                                           uint32_t *out, uint32_t *tmp) {
    constexpr int PER = SCAN_BLOCK / THREADS;
    uint32_t before = 0, base;
    for (uint64_t j = threadIdx.x; j < block; j += THREADS) before += part[j];
    block_excl_scan(before, tmp, &base);
    const uint64_t i0 = block * SCAN_BLOCK + (uint64_t)threadIdx.x * PER;
    uint32_t v[PER], x = 0;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        v[q] = i0 + q < m ? in[i0 + q] : 0u;
        x += v[q];
    }
    uint32_t total;
    uint32_t run = base + block_excl_scan(x, tmp, &total);
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        if (i0 + q < m) out[i0 + q] = run;
        run += v[q];
    }
    if (threadIdx.x == 0 && (block + 1) * SCAN_BLOCK >= m) out[m] = base + total;
}

// non-cold accesses of bucket b (t >> S == b), in tiles
__device__ __forceinline__ uint32_t bucket_tiles(const uint32_t *Zc, uint64_t n, int S, uint64_t b) {
    uint64_t lo = b << S, hi = (b + 1) << S;
    lo = lo < n ? lo : n;
    hi = hi < n ? hi : n;
    const uint64_t size = cnt_lt(hi, Zc) - cnt_lt(lo, Zc);
    return (uint32_t)((size + DOM_TILE - 1) / DOM_TILE);
}

// One bucket of a level: its first tile (the tiles of the buckets before it;
// there are at most a few thousand) and its tiles' entries in tile_bucket, so
// that the level's steps need one load instead of a search.
__device__ __forceinline__ void map_tiles(const uint32_t *Zc, uint64_t n, int S, uint64_t nbuckets, uint64_t b,
                                          uint32_t *tfirst, uint32_t *tile_bucket, uint32_t *tmp) {
    uint32_t before = 0, first;
    for (uint64_t j = threadIdx.x; j < b; j += blockDim.x) before += bucket_tiles(Zc, n, S, j);
    block_excl_scan(before, tmp, &first);
    const uint32_t mine = bucket_tiles(Zc, n, S, b);
    if (threadIdx.x == 0) {
        tfirst[b] = first;
        if (b + 1 == nbuckets) tfirst[nbuckets] = first + mine;
    }
    for (uint32_t j = threadIdx.x; j < mine; j += blockDim.x) tile_bucket[first + j] = (uint32_t)b;
}

// ---- one MSD level of the dominance count (8-bit digits of t) -----------
// Tiles: FIRST reads next[] in index order (= v order) in fixed index ranges,
// one bucket; later levels read the previous level's output with tiles that
// never straddle a bucket (bucket = t >> (s + k)), located through tfirst.
struct TileLoc {
    uint64_t bucket, e0, e1, first_tile;
    bool valid;
};

template <bool FIRST>
__device__ __forceinline__ TileLoc locate_tile(uint64_t tile, uint64_t n, const uint32_t *Zc,
                                               int S, const uint32_t *tfirst, uint64_t nbuckets,
                                               const uint32_t *tile_bucket) {
    TileLoc L{0, 0, 0, 0, true};
    if (FIRST) {
        const uint64_t tiles = (n + DOM_TILE - 1) / DOM_TILE;
        if (tile >= tiles) { L.valid = false; return L; }
        L.e0 = tile * DOM_TILE;
        L.e1 = L.e0 + DOM_TILE < n ? L.e0 + DOM_TILE : n;
        return L;
    }
    if (tile >= tfirst[nbuckets]) { L.valid = false; return L; }
    const uint64_t lo = tile_bucket[tile];
    L.bucket = lo;
    L.first_tile = tfirst[lo];
    uint64_t blo = lo << S, bhi = (lo + 1) << S;
    blo = blo < n ? blo : n;
    bhi = bhi < n ? bhi : n;
    const uint64_t bs = cnt_lt(blo, Zc), be = cnt_lt(bhi, Zc);
    L.e0 = bs + (tile - L.first_tile) * DOM_TILE;
    L.e1 = L.e0 + DOM_TILE < be ? L.e0 + DOM_TILE : be;
    return L;
}

template <bool FIRST>
__device__ __forceinline__ void load_tile(const TileLoc &L, const uint32_t *in_t,
                                          const uint32_t *in_acc, int w, int lane,
                                          uint32_t (&t)[DOM_CHUNKS_PER_WAVE], uint32_t (&acc)[DOM_CHUNKS_PER_WAVE],
                                          bool (&ok)[DOM_CHUNKS_PER_WAVE], bool want_acc) {
#pragma unroll
    for (int i = 0; i < DOM_CHUNKS_PER_WAVE; ++i) {
        const uint64_t e = L.e0 + (uint64_t)(w * DOM_CHUNKS_PER_WAVE + i) * WAVE + lane;
        if (FIRST) {
            const uint32_t x = e < L.e1 ? in_t[e] : NONE;
            ok[i] = x != NONE;
            t[i] = x;
            acc[i] = 0;
        } else {
            ok[i] = e < L.e1;
            t[i] = ok[i] ? in_t[e] : 0u;
            acc[i] = (ok[i] && want_acc) ? in_acc[e] : 0u;
        }
    }
}

// Per-tile digit counts (and whether the tile starts a bucket), the input of
// the segmented scan over tiles.  Only counts are needed here, so instead of
// ranking lanes each run of equal digits in a 64-lane chunk (runs are long at
// the top levels, where t grows with v) adds its length with one LDS atomic.
// A workgroup takes COUNT_TPW consecutive tiles and issues every lookup and
// load of all of them before counting: one tile's work is too short to
// cover the chain of dependent loads (tile -> bucket -> range -> elements).
constexpr int COUNT_TPW = 4;
template <bool FIRST>
__device__ __forceinline__ bool count_tiles(const uint32_t *in_t, uint64_t n, const uint32_t *Zc, int s, int k,
                                            const uint32_t *tfirst, uint64_t nbuckets, const uint32_t *tile_bucket,
                                            uint16_t *cnt, uint8_t *seg, uint64_t grp,
                                            uint32_t (*s_cnt)[DOM_RADIX]) {
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), w = tid / WAVE;
    __syncthreads();   // the previous group's counts are written out
    const uint64_t tile0 = grp * COUNT_TPW;
    // an invalid tile (past the level's last) has an empty range: it loads
    // nothing, and every later tile is invalid too
    TileLoc L[COUNT_TPW];
#pragma unroll
    for (int q = 0; q < COUNT_TPW; ++q)
        L[q] = locate_tile<FIRST>(tile0 + q, n, Zc, s + k, tfirst, nbuckets, tile_bucket);
    if (!L[0].valid) return false;   // every later group is past the level's last tile too
    for (int i = tid; i < COUNT_TPW * DOM_RADIX; i += DOM_THREADS) (&s_cnt[0][0])[i] = 0;
    uint32_t t[COUNT_TPW][DOM_CHUNKS_PER_WAVE], acc[DOM_CHUNKS_PER_WAVE];
    bool ok[COUNT_TPW][DOM_CHUNKS_PER_WAVE];
#pragma unroll
    for (int q = 0; q < COUNT_TPW; ++q) load_tile<FIRST>(L[q], in_t, nullptr, w, lane, t[q], acc, ok[q], false);
    __syncthreads();
    const uint32_t dmask = (1u << k) - 1u;
#pragma unroll
    for (int q = 0; q < COUNT_TPW; ++q) {
#pragma unroll
        for (int i = 0; i < DOM_CHUNKS_PER_WAVE; ++i) {
            // invalid lanes take digit RADIX (never counted) so they end runs
            const uint32_t d = ok[q][i] ? (t[q][i] >> s) & dmask : (uint32_t)DOM_RADIX;
            const uint32_t dl = from_lower(d);   // lane 0 keeps its own and is a head anyway
            const bool head = lane == 0 || dl != d;
            const uint64_t heads = ballot(head);
            // next head above this lane (or 64): the run is [lane, next)
            const uint64_t above = lane == WAVE - 1 ? 0ull : heads & (~0ull << (lane + 1));
            const uint32_t next = above ? (uint32_t)__builtin_ctzll(above) : (uint32_t)WAVE;
            if (head && d < (uint32_t)DOM_RADIX) atomicAdd(&s_cnt[q][d], next - (uint32_t)lane);
        }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < COUNT_TPW; ++q) {
        if (!L[q].valid) break;
        const uint64_t tile = tile0 + q;
        if (tid < DOM_RADIX) cnt[tile * DOM_RADIX + tid] = (uint16_t)s_cnt[q][tid];
        if (tid == 0) seg[tile] = FIRST ? (tile == 0) : (tile == L[q].first_tile);
    }
    return true;
}

// Segmented exclusive scan over tiles, per digit (a bucket's first tile
// restarts the sum), in three steps over groups of tiles.  A group's tiles are
// walked one after the other by one workgroup, so groups are small while there
// are few tiles (16 tiles up to 16,384; at 489 tiles the steps took 58 us each
// with groups of 256, two workgroups) and large enough afterwards that the
// carry handles them 1024 at a time.
constexpr int SEG_BATCH = 16;
constexpr uint64_t SEG_GROUP_MAX = 256;
static uint64_t seg_group(uint64_t tiles) {
    uint64_t g = (tiles + 1023) / 1024;
    g = (g + SEG_BATCH - 1) / SEG_BATCH * SEG_BATCH;
    return g < (uint64_t)SEG_BATCH ? (uint64_t)SEG_BATCH : g < SEG_GROUP_MAX ? g : SEG_GROUP_MAX;
}

__device__ __forceinline__ uint64_t total_tiles(const uint32_t *tfirst_end, uint64_t fixed) {
    return tfirst_end ? (uint64_t)*tfirst_end : fixed;
}

// A: per group (rows [r0, r1) of digit d), the sum after its last bucket start,
// and whether it has one
__device__ __forceinline__ void seg_reduce(const uint16_t *cnt, const uint8_t *seg, uint64_t r0, uint64_t r1, int d,
                                           uint64_t grp, uint32_t *gsum, uint8_t *ghas) {
    uint32_t tail = 0;
    bool has = false;
    for (uint64_t r = r0; r < r1; r += SEG_BATCH) {
        uint32_t c[SEG_BATCH];
        bool f[SEG_BATCH];
#pragma unroll
        for (int q = 0; q < SEG_BATCH; ++q) {
            const bool in = r + q < r1;
            c[q] = in ? cnt[(r + q) * DOM_RADIX + d] : 0u;
            f[q] = in && seg[r + q];
        }
#pragma unroll
        for (int q = 0; q < SEG_BATCH; ++q) {
            if (f[q]) { tail = 0; has = true; }
            tail += c[q];
        }
    }
    gsum[grp * DOM_RADIX + d] = tail;
    if (d == 0) ghas[grp] = has;
}

// B: carry into every group: per digit (one workgroup each), a segmented
// scan over the groups where a group holding a bucket start restarts the
// sum.  Inside a wave: the plain prefix sum minus the sum before the last
// start at or below the lane (found with a ballot); across the waves of a
// workgroup's chunk of groups and across chunks: a short serial carry.
constexpr int CARRY_WAVES_MAX = 16;
__device__ __forceinline__ void seg_carry(const uint32_t *gsum, const uint8_t *ghas, uint64_t groups, int d,
                                          uint32_t *gin, uint32_t *s_val, uint32_t *s_has) {
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), w = tid / WAVE, nw = (int)blockDim.x / WAVE;
    uint32_t carry = 0;   // carry into the current chunk
    for (uint64_t g0 = 0; g0 < groups; g0 += blockDim.x) {
        const uint64_t g = g0 + tid;
        const bool in = g < groups;
        const bool f = in && ghas[g];
        const uint32_t v = in ? gsum[g * DOM_RADIX + d] : 0u;
        const uint32_t S = wave_incl_scan(v);
        const uint64_t fm = ballot(f);
        const uint64_t le = fm & (lane == WAVE - 1 ? ~0ull : ((2ull << lane) - 1));   // starts at or below me
        const int last = le ? 63 - __builtin_clzll(le) : -1;
        const uint32_t before = (uint32_t)__shfl((int)S, last > 0 ? last - 1 : 0, WAVE);
        const uint32_t seg = last > 0 ? S - before : S;   // sum since the last start (or since lane 0)
        if (lane == WAVE - 1) {
            s_val[w] = seg;
            s_has[w] = fm != 0;
        }
        __syncthreads();
        uint32_t cin = carry;   // carry into this wave
        for (int x = 0; x < w; ++x) cin = s_has[x] ? s_val[x] : cin + s_val[x];
        uint32_t chunk_out = cin;
        for (int x = w; x < nw; ++x) chunk_out = s_has[x] ? s_val[x] : chunk_out + s_val[x];
        const uint32_t incl = last >= 0 ? seg : cin + seg;   // carry after group g
        const uint32_t prev = (uint32_t)__shfl_up((int)incl, 1, WAVE);
        if (in) gin[g * DOM_RADIX + d] = lane == 0 ? cin : prev;
        carry = chunk_out;
        __syncthreads();
    }
}

// C: per group, the exclusive prefix of every tile
__device__ __forceinline__ void seg_scan(const uint16_t *cnt, const uint8_t *seg, uint64_t r0, uint64_t r1, int d,
                                         uint64_t grp, const uint32_t *gin, uint32_t *pre) {
    uint32_t run = gin[grp * DOM_RADIX + d];
    for (uint64_t r = r0; r < r1; r += SEG_BATCH) {
        uint32_t c[SEG_BATCH];
        bool f[SEG_BATCH];
#pragma unroll
        for (int q = 0; q < SEG_BATCH; ++q) {
            const bool in = r + q < r1;
            c[q] = in ? cnt[(r + q) * DOM_RADIX + d] : 0u;
            f[q] = in && seg[r + q];
        }
#pragma unroll
        for (int q = 0; q < SEG_BATCH; ++q) {
            if (r + q < r1) {
                if (f[q]) run = 0;
                pre[(r + q) * DOM_RADIX + d] = run;
                run += c[q];
            }
        }
    }
}

// The level itself: per tile, every element adds the number of earlier
// elements of its bucket (in v order) with a smaller digit -- from earlier
// tiles (the scanned counts), earlier chunks of the tile (2-D prefix over
// (chunk, digit) in LDS) and earlier lanes of its chunk (ballot masks) --
// and the tile is written out digit-partitioned through LDS.
// LDS of the level: chunk histograms -> column prefix (h); once every position
// is known, the staged tile (t, then acc) in the same space: 36 KB in all, so
// four workgroups share a CU.
struct DomLds {
    uint16_t h[DOM_CHUNKS][DOM_RADIX];
    uint16_t pl[DOM_CHUNKS][DOM_RADIX];    // 2-D prefix (earlier chunks, smaller digit)
    // per-digit tile starts and smaller-digit counts; before that, the two
    // half sums of the column prefix
    uint32_t part[2][DOM_RADIX];
    uint32_t base[DOM_RADIX];
    uint32_t tmp[DOM_WAVES];
};
static_assert(sizeof(DomLds::h) >= 2 * DOM_TILE * sizeof(uint32_t), "the stage fits the histograms");

template <bool FIRST>
__device__ __forceinline__ bool dominance_tile(DomLds &D, const uint32_t *in_t, const uint32_t *in_acc,
                                               uint32_t *out_t, uint32_t *out_acc, uint64_t n, const uint32_t *Zc,
                                               int s, int k, const uint32_t *tfirst, uint64_t nbuckets,
                                               const uint32_t *tile_bucket, const uint32_t *pre, int32_t *err,
                                               uint64_t tile) {
    uint16_t(*s_h)[DOM_RADIX] = D.h;
    uint16_t(*s_pl)[DOM_RADIX] = D.pl;
    uint32_t(*s_part)[DOM_RADIX] = D.part;
    uint32_t *s_base = D.base, *s_tmp = D.tmp;
    uint32_t *s_st = reinterpret_cast<uint32_t *>(&s_h[0][0]);   // staged t
    uint32_t *s_sa = s_st + DOM_TILE;                           // staged acc
    uint32_t *s_lstart = s_part[0], *s_gl = s_part[1];
    // (an opaque copy: in a loop over tiles what is derived from it is worked
    // out per tile instead of being held across the loop)
    int tid = threadIdx.x;
    __asm__ volatile("" : "+v"(tid));
    const int lane = tid & (WAVE - 1);
    const int w = tid / WAVE;
    const uint32_t dmask = (1u << k) - 1u;
    __syncthreads();   // the previous tile has left the LDS
    const TileLoc L = locate_tile<FIRST>(tile, n, Zc, s + k, tfirst, nbuckets, tile_bucket);
    if (!L.valid) return false;   // every later tile is past the level's last too
    // same digit, earlier tiles of the bucket (threads below RADIX own a digit)
    const uint32_t G = tid < DOM_RADIX ? pre[tile * DOM_RADIX + tid] : 0u;
    {
        uint64_t *z = reinterpret_cast<uint64_t *>(&s_h[0][0]);
        for (int i = tid; i < DOM_CHUNKS * DOM_RADIX / 4; i += DOM_THREADS) z[i] = 0;
    }
    uint32_t t[DOM_CHUNKS_PER_WAVE], acc[DOM_CHUNKS_PER_WAVE];
    bool ok[DOM_CHUNKS_PER_WAVE];
    load_tile<FIRST>(L, in_t, in_acc, w, lane, t, acc, ok, true);
    __syncthreads();

    // ---- rank inside each 64-lane chunk
    uint16_t q_ic[DOM_CHUNKS_PER_WAVE], l_ic[DOM_CHUNKS_PER_WAVE];
#pragma unroll
    for (int i = 0; i < DOM_CHUNKS_PER_WAVE; ++i) {
        const int c = w * DOM_CHUNKS_PER_WAVE + i;
        const uint32_t d = (t[i] >> s) & dmask;
        uint32_t lt;
        // the top level often has few digit bits (8 buckets at 2^31 accesses)
        const uint64_t eq = k <= 4 ? rank_digit<4>(d, ballot(ok[i]), &lt) : rank_digit<8>(d, ballot(ok[i]), &lt);
        q_ic[i] = ok[i] ? (uint16_t)mbcnt(eq) : 0;
        l_ic[i] = ok[i] ? (uint16_t)lt : 0;
        if (ok[i] && q_ic[i] == 0) s_h[c][d] = (uint16_t)__popcll(eq);
    }
    __syncthreads();

    // ---- column prefix over chunks (thread = digit, two halves of the
    // chunks) and tile totals; all loads are issued before any store
    uint32_t tot = 0;
    {
        constexpr int HALF = DOM_CHUNKS / 2;
        const int d = tid & (DOM_RADIX - 1), c0 = (tid / DOM_RADIX) * HALF;
        uint16_t h[HALF];
        uint32_t sum = 0;
#pragma unroll
        for (int c = 0; c < HALF; ++c) {
            h[c] = s_h[c0 + c][d];
            sum += h[c];
        }
        s_part[tid / DOM_RADIX][d] = sum;
        __syncthreads();
        uint32_t run = c0 ? s_part[0][d] : 0u;
        tot = tid < DOM_RADIX ? s_part[0][d] + s_part[1][d] : 0u;
#pragma unroll
        for (int c = 0; c < HALF; ++c) {
            s_h[c0 + c][d] = (uint16_t)run;
            run += h[c];
        }
    }
    __syncthreads();
    // ---- row prefix over digits: s_pl[c][d] = sum_{d' < d} s_h[c][d']
    for (int c = w * (DOM_CHUNKS / DOM_WAVES); c < (w + 1) * (DOM_CHUNKS / DOM_WAVES); ++c) {
        const uint32_t a0 = s_h[c][4 * lane + 0], a1 = s_h[c][4 * lane + 1];
        const uint32_t a2 = s_h[c][4 * lane + 2], a3 = s_h[c][4 * lane + 3];
        const uint32_t x = wave_excl_scan(a0 + a1 + a2 + a3);
        s_pl[c][4 * lane + 0] = (uint16_t)x;
        s_pl[c][4 * lane + 1] = (uint16_t)(x + a0);
        s_pl[c][4 * lane + 2] = (uint16_t)(x + a0 + a1);
        s_pl[c][4 * lane + 3] = (uint16_t)(x + a0 + a1 + a2);
    }
    uint32_t n_valid;
    const uint32_t lst = block_excl_scan(tot, s_tmp, &n_valid);
    uint32_t gsum;
    const uint32_t GL = block_excl_scan(G, s_tmp, &gsum);   // smaller digit, earlier tiles
    if (tid < DOM_RADIX) {
        const uint64_t X = ((L.bucket << k) + (uint64_t)tid) << s;
        const uint64_t sub = cnt_lt(X < n ? X : n, Zc);
        s_lstart[tid] = lst;
        s_gl[tid] = GL;
        s_base[tid] = (uint32_t)(sub + G - lst);   // wraps mod 2^32 like positions
    }
    __syncthreads();

    // ---- stage the tile digit-partitioned, with the level's count added
    uint32_t pj[DOM_CHUNKS_PER_WAVE];
#pragma unroll
    for (int i = 0; i < DOM_CHUNKS_PER_WAVE; ++i) {
        if (ok[i]) {
            const int c = w * DOM_CHUNKS_PER_WAVE + i;
            const uint32_t d = (t[i] >> s) & dmask;
            pj[i] = s_lstart[d] + s_h[c][d] + q_ic[i];
            acc[i] += s_gl[d] + s_pl[c][d] + l_ic[i];
        }
    }
    __syncthreads();   // the histograms are read: their space becomes the stage
#pragma unroll
    for (int i = 0; i < DOM_CHUNKS_PER_WAVE; ++i) {
        if (ok[i]) {
            s_st[pj[i]] = t[i];
            s_sa[pj[i]] = acc[i];
        }
    }
    __syncthreads();
    for (uint32_t j = tid; j < n_valid; j += DOM_THREADS) {
        const uint32_t tt = s_st[j];
        const uint32_t d = (tt >> s) & dmask;
        const uint32_t dst = s_base[d] + j;
        // consistent prev/next always land inside; inconsistent input is
        // reported instead of written out of bounds
        if (dst < n) {
            out_t[dst] = tt;
            out_acc[dst] = s_sa[j];
        } else {
            atomicOr(err, DEV_ERR_BAD_LAYOUT);
        }
    }
    return true;
}

// Last 12 bits, one workgroup per 4096-range of t, then D in t order.  The
// level-A counts go straight into a slot per t (acc included), so only the
// six low bits of t are staged for level B, and the prev values needed at the
// end are loaded up front; LDS stays under 40 KB (four workgroups per CU).
struct LocalLds {
    uint32_t slot[LOCAL_SPAN];           // by t: acc + counts; first the column-prefix sums
    uint16_t h[LOC_CHUNKS][64];          // chunk histograms -> column prefix
    uint16_t pl[LOC_CHUNKS][64];         // 2-D prefix (earlier chunks, smaller digit)
    uint8_t low[LOCAL_SPAN];             // bits 0..5 of t, grouped by bits 6..11
    uint32_t lstart[65];
    uint32_t tmp[LOC_WAVES];
};
__device__ __forceinline__ void local_range(LocalLds &D, const uint32_t *in_t, const uint32_t *in_acc,
                                            const uint32_t *prev, uint64_t n, const uint32_t *Zc, uint32_t *dist,
                                            uint64_t chunk) {
    uint32_t *slot = D.slot, *s_lstart = D.lstart, *s_tmp = D.tmp;
    uint16_t(*s_h)[64] = D.h;
    uint16_t(*s_pl)[64] = D.pl;
    uint8_t *s_low = D.low;
    uint32_t(*s_part)[64] = reinterpret_cast<uint32_t(*)[64]>(slot);   // [LOC_PARTS][64]

    int tid = threadIdx.x;
    __asm__ volatile("" : "+v"(tid));
    const int lane = tid & (WAVE - 1);
    const int w = tid / WAVE;
    __syncthreads();   // the previous range has left the LDS
    const uint64_t r0 = chunk * LOCAL_SPAN;
    const uint64_t r1 = r0 + LOCAL_SPAN < n ? r0 + LOCAL_SPAN : n;
    const uint64_t e0 = cnt_lt(r0, Zc), e1 = cnt_lt(r1, Zc);
    for (int i = tid; i < LOC_CHUNKS * 64 / 2; i += LOC_THREADS) reinterpret_cast<uint32_t *>(&s_h[0][0])[i] = 0;

    // ---- loads: the range's elements (v order) and its prev values (t order)
    constexpr int PER = LOCAL_SPAN / LOC_THREADS;   // 8
    // (32-bit offsets from per-range base pointers)
    uint32_t t[LOC_CPW], acc[LOC_CPW], p[PER];
    bool ok[LOC_CPW];
    const uint32_t ne = (uint32_t)(e1 - e0), nt = (uint32_t)(r1 - r0);
    const uint32_t *tb = in_t + e0, *ab = in_acc + e0, *pb = prev + r0;
#pragma unroll
    for (int i = 0; i < LOC_CPW; ++i) {
        const uint32_t o = (uint32_t)((w * LOC_CPW + i) * WAVE + lane);
        ok[i] = o < ne;
        const uint32_t oc = ok[i] ? o : 0u;
        t[i] = tb[oc];
        acc[i] = ab[oc];
    }
    const uint32_t tofs = (uint32_t)tid * PER;
    const uint64_t tbase = r0 + tofs;
    // a full range with aligned bases moves prev and D as two 16-byte
    // vectors per thread
    const bool vec = nt == LOCAL_SPAN && ((reinterpret_cast<uintptr_t>(pb) | reinterpret_cast<uintptr_t>(dist + r0)) & 15) == 0;
    static_assert(PER == 8, "two 16-byte vectors per thread");
    if (vec) {
        const uint4 a = reinterpret_cast<const uint4 *>(pb + tofs)[0];
        const uint4 b = reinterpret_cast<const uint4 *>(pb + tofs)[1];
        p[0] = a.x; p[1] = a.y; p[2] = a.z; p[3] = a.w;
        p[4] = b.x; p[5] = b.y; p[6] = b.z; p[7] = b.w;
    } else {
#pragma unroll
        for (int j = 0; j < PER; ++j) p[j] = pb[tofs + j < nt ? tofs + j : 0u];
    }
    __syncthreads();   // chunk histograms zeroed

    // ---- level A: digit = bits 6..11 of t, chunks of 64 in v order
    uint8_t qa[LOC_CPW], la[LOC_CPW];
#pragma unroll
    for (int i = 0; i < LOC_CPW; ++i) {
        const int c = w * LOC_CPW + i;
        const uint32_t d = (t[i] >> 6) & 63;
        uint32_t lt;
        const uint64_t eq = rank_digit<6>(d, ballot(ok[i]), &lt);
        qa[i] = ok[i] ? (uint8_t)mbcnt(eq) : 0;
        la[i] = ok[i] ? (uint8_t)lt : 0;
        if (ok[i] && qa[i] == 0) s_h[c][d] = (uint16_t)__popcll(eq);
    }
    __syncthreads();
    // column prefix: thread (digit d, part q) scans LOC_CHUNKS / LOC_PARTS
    // chunks, then the part sums are combined
    {
        constexpr int CP = LOC_CHUNKS / LOC_PARTS;
        const int d = tid & 63, q = tid >> 6;
        uint16_t h[CP];
        uint32_t sum = 0;
#pragma unroll
        for (int c = 0; c < CP; ++c) {
            h[c] = s_h[q * CP + c][d];
            sum += h[c];
        }
        s_part[q][d] = sum;
        __syncthreads();
        uint32_t run = 0, tot = 0;
#pragma unroll
        for (int x = 0; x < LOC_PARTS; ++x) {
            const uint32_t v = s_part[x][d];
            if (x < q) run += v;
            tot += v;
        }
#pragma unroll
        for (int c = 0; c < CP; ++c) {
            s_h[q * CP + c][d] = (uint16_t)run;
            run += h[c];
        }
        if (q == 0) {
            const uint32_t incl = wave_incl_scan(tot);
            s_lstart[d] = incl - tot;
            if (d == 63) s_lstart[64] = incl;
        }
    }
    __syncthreads();
    for (int c = w * LOC_CPW; c < (w + 1) * LOC_CPW; ++c) s_pl[c][lane] = (uint16_t)wave_excl_scan(s_h[c][lane]);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < LOC_CPW; ++i) {
        if (ok[i]) {
            const int c = w * LOC_CPW + i;
            const uint32_t d = (t[i] >> 6) & 63;
            s_low[s_lstart[d] + s_h[c][d] + qa[i]] = (uint8_t)(t[i] & 63);
            slot[t[i] & (LOCAL_SPAN - 1)] = acc[i] + s_pl[c][d] + la[i];
        }
    }
    __syncthreads();

    // ---- level B: bits 0..5 inside each 64-range (at most 64 elements,
    // all with different t, so their six low bits are distinct)
    for (int g = w; g < 64; g += LOC_WAVES) {
        const uint32_t base = s_lstart[g];
        const bool okb = (uint32_t)lane < s_lstart[g + 1] - base;
        const uint32_t lb = okb ? s_low[base + lane] : 0u;
        const uint32_t lt = count_smaller_distinct6(lb, okb);
        if (okb) slot[g * 64 + lb] += lt;
    }
    __syncthreads();

    // ---- D in t order: Z(t) from a block scan of cold flags
    uint32_t cold = 0;
#pragma unroll
    for (int j = 0; j < PER; ++j) cold += (tbase + j < n && p[j] == NONE) ? 1u : 0u;
    uint32_t allcold;
    uint32_t z = Zc[chunk] + block_excl_scan(cold, s_tmp, &allcold);
    uint32_t dv[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        if (p[j] == NONE) {
            dv[j] = NONE;
            ++z;
        } else {
            dv[j] = z + slot[(tofs + j) & (LOCAL_SPAN - 1)] - (p[j] + 1u);
        }
    }
    if (vec) {
        reinterpret_cast<uint4 *>(dist + tbase)[0] = make_uint4(dv[0], dv[1], dv[2], dv[3]);
        reinterpret_cast<uint4 *>(dist + tbase)[1] = make_uint4(dv[4], dv[5], dv[6], dv[7]);
    } else {
#pragma unroll
        for (int j = 0; j < PER; ++j)
            if (tbase + j < n) dist[tbase + j] = dv[j];
    }
}

// ---- one launch per step
__global__ __launch_bounds__(256) void sd_cold_count_kernel(const uint32_t *__restrict__ prev, uint64_t n,
                                                            uint32_t *__restrict__ cnt, int32_t *__restrict__ hdr, const int32_t *gate) {
    if (gated_off(gate)) return;
    __shared__ uint32_t tmp[4];
    if (hdr && blockIdx.x == 0 && threadIdx.x == 0) *hdr = 0;   // the call's status
    const uint64_t nchunks = (n + LOCAL_SPAN - 1) / LOCAL_SPAN;
    for (uint64_t c = blockIdx.x; c < nchunks; c += gridDim.x) cold_count<256>(prev, n, c, cnt, tmp);
}
__global__ __launch_bounds__(SCAN_THREADS) void sd_scan_reduce_kernel(const uint32_t *__restrict__ in, uint64_t m,
                                                                      uint32_t *__restrict__ part, const int32_t *gate) {
    if (gated_off(gate)) return;
    __shared__ uint32_t tmp[SCAN_THREADS / WAVE];
    scan_reduce(in, m, blockIdx.x, part, tmp);
}
__global__ __launch_bounds__(SCAN_THREADS) void sd_scan_apply_kernel(const uint32_t *__restrict__ in, uint64_t m,
                                                                     const uint32_t *__restrict__ part,
                                                                     uint32_t *__restrict__ out, const int32_t *gate) {
    if (gated_off(gate)) return;
    __shared__ uint32_t tmp[SCAN_THREADS / WAVE];
    scan_apply<SCAN_THREADS>(in, m, blockIdx.x, part, out, tmp);
}
__global__ __launch_bounds__(256) void sd_tile_map_kernel(const uint32_t *__restrict__ Zc, uint64_t n, int S,
                                                          uint64_t nbuckets, uint32_t *__restrict__ tfirst,
                                                          uint32_t *__restrict__ tile_bucket, const int32_t *gate) {
    if (gated_off(gate)) return;
    __shared__ uint32_t tmp[4];
    map_tiles(Zc, n, S, nbuckets, blockIdx.x, tfirst, tile_bucket, tmp);
}
template <bool FIRST>
__global__ __launch_bounds__(DOM_THREADS) void sd_count_kernel(
    const uint32_t *__restrict__ in_t, uint64_t n, const uint32_t *__restrict__ Zc, int s, int k,
    const uint32_t *__restrict__ tfirst, uint64_t nbuckets, const uint32_t *__restrict__ tile_bucket,
    uint16_t *__restrict__ cnt, uint8_t *__restrict__ seg, uint64_t groups, const int32_t *gate) {
    if (gated_off(gate)) return;
    __shared__ uint32_t s_cnt[COUNT_TPW][DOM_RADIX];
    for (uint64_t grp = blockIdx.x; grp < groups; grp += gridDim.x)
        if (!count_tiles<FIRST>(in_t, n, Zc, s, k, tfirst, nbuckets, tile_bucket, cnt, seg, grp, s_cnt)) break;
}
__global__ __launch_bounds__(DOM_RADIX) void sd_seg_reduce_kernel(const uint16_t *__restrict__ cnt,
                                                                  const uint8_t *__restrict__ seg,
                                                                  const uint32_t *tfirst_end, uint64_t fixed,
                                                                  uint64_t group, uint32_t *__restrict__ gsum,
                                                                  uint8_t *__restrict__ ghas, const int32_t *gate) {
    if (gated_off(gate)) return;
    const uint64_t rows = total_tiles(tfirst_end, fixed), r0 = blockIdx.x * group;
    if (r0 < rows)
        seg_reduce(cnt, seg, r0, r0 + group < rows ? r0 + group : rows, threadIdx.x, blockIdx.x, gsum, ghas);
}
__global__ __launch_bounds__(CARRY_WAVES_MAX *WAVE) void sd_seg_carry_kernel(const uint32_t *__restrict__ gsum,
                                                                             const uint8_t *__restrict__ ghas,
                                                                             const uint32_t *tfirst_end,
                                                                             uint64_t fixed, uint64_t group,
                                                                             uint32_t *__restrict__ gin, const int32_t *gate) {
    if (gated_off(gate)) return;
    __shared__ uint32_t s_val[CARRY_WAVES_MAX], s_has[CARRY_WAVES_MAX];
    const uint64_t rows = total_tiles(tfirst_end, fixed);
    seg_carry(gsum, ghas, (rows + group - 1) / group, blockIdx.x, gin, s_val, s_has);
}
__global__ __launch_bounds__(DOM_RADIX) void sd_seg_scan_kernel(const uint16_t *__restrict__ cnt,
                                                                const uint8_t *__restrict__ seg,
                                                                const uint32_t *tfirst_end, uint64_t fixed,
                                                                uint64_t group, const uint32_t *__restrict__ gin,
                                                                uint32_t *__restrict__ pre, const int32_t *gate) {
    if (gated_off(gate)) return;
    const uint64_t rows = total_tiles(tfirst_end, fixed), r0 = blockIdx.x * group;
    if (r0 < rows)
        seg_scan(cnt, seg, r0, r0 + group < rows ? r0 + group : rows, threadIdx.x, blockIdx.x, gin, pre);
}
template <bool FIRST>
__global__ __launch_bounds__(DOM_THREADS) void sd_dominance_kernel(
    const uint32_t *__restrict__ in_t, const uint32_t *__restrict__ in_acc, uint32_t *__restrict__ out_t,
    uint32_t *__restrict__ out_acc, uint64_t n, const uint32_t *__restrict__ Zc, int s, int k,
    const uint32_t *__restrict__ tfirst, uint64_t nbuckets, const uint32_t *__restrict__ tile_bucket,
    const uint32_t *__restrict__ pre, int32_t *__restrict__ err, uint64_t ntiles, const int32_t *gate) {
    if (gated_off(gate)) return;
    __shared__ DomLds D;
    for (uint64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x)
        if (!dominance_tile<FIRST>(D, in_t, in_acc, out_t, out_acc, n, Zc, s, k, tfirst, nbuckets, tile_bucket, pre,
                                   err, tile))
            break;
}
__global__ __launch_bounds__(LOC_THREADS, 6) void sd_local_kernel(
    const uint32_t *__restrict__ in_t, const uint32_t *__restrict__ in_acc, const uint32_t *__restrict__ prev,
    uint64_t n, const uint32_t *__restrict__ Zc, uint32_t *__restrict__ dist, const int32_t *gate) {
    if (gated_off(gate)) return;
    __shared__ LocalLds D;
    const uint64_t nchunks = (n + LOCAL_SPAN - 1) / LOCAL_SPAN;
    for (uint64_t chunk = blockIdx.x; chunk < nchunks; chunk += gridDim.x)
        local_range(D, in_t, in_acc, prev, n, Zc, dist, chunk);
}

// ---- request-level residency --------------------------------------------
// Request-level distance from the per-access distance of the request-ordered
// stream.  With v = prev + 1 (0 for a cold access) and t in request [s, e):
//     dist_req(t) = dist(t) - #{ j in [s, t) : v(j) < v(t) }.
// When v(t) exceeds every earlier v of its request the count is t - s.  That
// is always so for chained prefix keys: a block's last use is no later than
// the last use of any shallower block of its chain, and each request lists
// its shallower blocks after its deeper ones.  Other key streams take a
// direct count over [s, t) for the accesses that break the order.
// One wave per request (grid-stride), REQ_ITEMS x 64 accesses per step.  Bound:
// the reads of prev and dist, now that a step's are under way during the one
// before (6.0e7 accesses 0.168 ms, 4.3 TB/s; loaded step by step in workgroups
// of four waves 0.318).
constexpr int REQ_ITEMS = 8;

// AHEAD: for long requests, whole steps with the next one's loads on their way.
template <bool AHEAD>
__global__ __launch_bounds__(256) void req_dist_kernel(const uint32_t *__restrict__ prev,
                                                       const uint32_t *__restrict__ dist,
                                                       const uint64_t *__restrict__ blk_off, uint32_t n_seqs,
                                                       uint64_t n, uint32_t *__restrict__ dist_req,
                                                       int32_t *__restrict__ err) {
    const int lane = threadIdx.x & (WAVE - 1);
    const uint32_t waves = gridDim.x * (blockDim.x / WAVE);
    const uint32_t w0 = __builtin_amdgcn_readfirstlane(blockIdx.x * (blockDim.x / WAVE) + threadIdx.x / WAVE);
    if (w0 == 0 && lane == 0 && (blk_off[0] != 0 || blk_off[n_seqs] != n)) atomicOr(err, DEV_ERR_BAD_LAYOUT);
    for (uint32_t r = w0; r < n_seqs; r += waves) {
        const uint64_t s = blk_off[r], e = blk_off[r + 1];
        if (s > e || e > n) {
            if (lane == 0) atomicOr(err, DEV_ERR_BAD_LAYOUT);
            continue;
        }
        uint32_t carry = 0;   // max v over the request's accesses before this step
        uint32_t v[REQ_ITEMS], d[REQ_ITEMS];
        auto step = [&](uint64_t base) {
#pragma unroll
            for (int i = 0; i < REQ_ITEMS; ++i) {
                const uint64_t t = base + i * WAVE + lane;
                // v(t) is above every earlier v iff it is the prefix max and
                // above the carry (earlier non-zero v are distinct from it)
                const uint32_t incl = wave_incl_max(v[i]);
                const bool top = v[i] == incl && v[i] > carry;
                carry = max(carry, (uint32_t)__builtin_amdgcn_readlane((int)incl, WAVE - 1));
                if (t >= e) continue;
                if (v[i] == 0u) {
                    dist_req[t] = NONE;
                } else if (top) {
                    dist_req[t] = d[i] - (uint32_t)(t - s);
                } else {
                    uint32_t c = 0;
                    for (uint64_t j = s; j < t; ++j) c += (prev[j] + 1u < v[i]) ? 1u : 0u;
                    dist_req[t] = d[i] - c;
                }
            }
        };
        uint64_t base = s;
        if (AHEAD && e - s >= REQ_ITEMS * WAVE) {
            uint32_t pn[REQ_ITEMS], dn[REQ_ITEMS];
            auto fetch = [&](uint64_t at) {
#pragma unroll
                for (int i = 0; i < REQ_ITEMS; ++i) {
                    pn[i] = prev[at + i * WAVE + lane];
                    dn[i] = dist[at + i * WAVE + lane];
                }
            };
            fetch(base);
            for (; e - base >= REQ_ITEMS * WAVE; base += REQ_ITEMS * WAVE) {
#pragma unroll
                for (int i = 0; i < REQ_ITEMS; ++i) {
                    v[i] = pn[i] + 1u;
                    d[i] = dn[i];
                }
                if (e - base >= 2 * REQ_ITEMS * WAVE) fetch(base + REQ_ITEMS * WAVE);
                step(base);
            }
        }
        for (; base < e; base += REQ_ITEMS * WAVE) {
#pragma unroll
            for (int i = 0; i < REQ_ITEMS; ++i) {
                const uint64_t t = base + i * WAVE + lane;
                const bool ok = t < e;
                v[i] = ok ? prev[t] + 1u : 0u;
                d[i] = ok ? dist[t] : 0u;
            }
            step(base);
        }
    }
}

// Each request's accesses in reverse (deepest block first): the recency
// order of request-level residency.  One wave per request, grid-stride.
__global__ __launch_bounds__(256) void req_order_kernel(const uint64_t *__restrict__ keys,
                                                        const uint32_t *__restrict__ depth,
                                                        const uint64_t *__restrict__ blk_off, uint32_t n_seqs,
                                                        uint64_t n, uint64_t *__restrict__ keys_out,
                                                        uint32_t *__restrict__ depth_out,
                                                        int32_t *__restrict__ err) {
    const int lane = threadIdx.x & (WAVE - 1);
    const uint64_t waves = (uint64_t)gridDim.x * (blockDim.x / WAVE);
    for (uint64_t r = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) / WAVE; r < n_seqs; r += waves) {
        const uint64_t a = blk_off[r], b = blk_off[r + 1];
        if (a > b || b > n) {
            if (lane == 0) atomicOr(err, DEV_ERR_BAD_LAYOUT);
            continue;
        }
        const uint64_t m = b - a;
        for (uint64_t j = lane; j < m; j += WAVE) {
            keys_out[b - 1 - j] = keys[a + j];
            if (depth) depth_out[b - 1 - j] = depth[a + j];
        }
    }
}

struct SdPlan {
    int passes;
    int s[4], k[4];
    uint64_t nbuckets[4];
    uint64_t grid[4];
    uint64_t max_buckets, max_grid;
};

static SdPlan plan_sd(uint64_t n) {
    SdPlan p{};
    int nbits = 0;
    while (nbits < 64 && (1ull << nbits) < n) ++nbits;   // bits of n-1
    const int g = nbits > LOCAL_BITS ? nbits - LOCAL_BITS : 0;
    p.passes = g == 0 ? 1 : (g + 7) / 8;
    if (g == 0) {
        p.k[0] = 1;
    } else {
        p.k[0] = g - 8 * (p.passes - 1);
        for (int i = 1; i < p.passes; ++i) p.k[i] = 8;
    }
    p.s[p.passes - 1] = LOCAL_BITS;
    for (int i = p.passes - 2; i >= 0; --i) p.s[i] = p.s[i + 1] + p.k[i + 1];
    p.max_buckets = 1;
    p.max_grid = 1;
    for (int i = 0; i < p.passes; ++i) {
        const int S = p.s[i] + p.k[i];
        p.nbuckets[i] = S >= 64 ? 1 : (n + (1ull << S) - 1) >> S;
        if (p.nbuckets[i] == 0) p.nbuckets[i] = 1;
        p.grid[i] = (n + DOM_TILE - 1) / DOM_TILE + (i == 0 ? 0 : p.nbuckets[i]);
        if (p.grid[i] == 0) p.grid[i] = 1;
        if (p.nbuckets[i] > p.max_buckets) p.max_buckets = p.nbuckets[i];
        if (p.grid[i] > p.max_grid) p.max_grid = p.grid[i];
    }
    return p;
}


struct SdWs {
    int32_t *hdr;
    uint32_t *cold, *Zc, *part, *tfirst;
    uint32_t *at, *aa, *bt, *ba;
    uint16_t *cnt;
    uint8_t *seg, *ghas;
    uint32_t *gsum, *gin, *pre, *tile_bucket;
    size_t bytes;
};

// workspace of one call
static SdWs carve_sd(void *ws, uint64_t n, const SdPlan &p) {
    Carver c{(char *)ws, 0};
    SdWs w;
    const uint64_t nchunks = (n + LOCAL_SPAN - 1) / LOCAL_SPAN;
    uint64_t groups = 1;
    for (int i = 0; i < p.passes; ++i) {
        const uint64_t g = (p.grid[i] + seg_group(p.grid[i]) - 1) / seg_group(p.grid[i]);
        if (g > groups) groups = g;
    }
    w.hdr = c.take<int32_t>(WS_HEADER / sizeof(int32_t));
    w.cold = c.take<uint32_t>(nchunks + 1);
    w.Zc = c.take<uint32_t>(nchunks + 2);
    const uint64_t nblocks = (nchunks + SCAN_BLOCK - 1) / SCAN_BLOCK;
    w.part = c.take<uint32_t>(nblocks + 1);
    w.tfirst = c.take<uint32_t>(p.max_buckets + 2);
    w.at = c.take<uint32_t>(n);
    w.aa = c.take<uint32_t>(n);
    w.bt = c.take<uint32_t>(n);
    w.ba = c.take<uint32_t>(n);
    w.cnt = c.take<uint16_t>(p.max_grid * DOM_RADIX);
    w.seg = c.take<uint8_t>(p.max_grid);
    w.ghas = c.take<uint8_t>(groups);
    w.gsum = c.take<uint32_t>(DOM_RADIX);
    w.gin = c.take<uint32_t>(DOM_RADIX);
    w.pre = c.take<uint32_t>(p.max_grid * DOM_RADIX);
    w.tile_bucket = c.take<uint32_t>(p.max_grid);
    w.bytes = c.off;
    return w;
}

// A level's group sums and carries: with more than one group they lie in the
// level's output acc array, which is written only after they are used (there
// are at least 4096 accesses then, and 32 per word needed).
struct SegSpace {
    uint32_t *gsum, *gin;
};
__host__ __device__ inline SegSpace seg_space(const SdWs &w, uint32_t *out_acc, uint64_t groups) {
    if (groups <= 1) return SegSpace{w.gsum, w.gin};
    return SegSpace{out_acc, out_acc + groups * DOM_RADIX};
}

// Workgroups per CU of the loops over tiles: enough that each takes only a
// few tiles (one tile per workgroup balances best: a static share of many
// tiles ran the dominance passes 25% slower).
constexpr int SD_GRID_PER_CU = 64;

// The dominance count, one launch per step, each gated; errors go to *err
// (nullptr: the workspace header, cleared here).
static pc_status stack_distance_steps(const uint32_t *prev, const uint32_t *next, uint64_t n, uint32_t *dist,
                                      void *ws, hipStream_t s, const int32_t *gate, int32_t *err) {
    const SdPlan p = plan_sd(n);
    const SdWs w = carve_sd(ws, n, p);
    if (n == 0) return fill_u32(reinterpret_cast<uint32_t *>(w.hdr), 0u, 1, s);
    // Z at every multiple of 4096 from the cold (prev = none) flags
    const uint64_t nchunks = (n + LOCAL_SPAN - 1) / LOCAL_SPAN;
    const uint64_t nblocks = (nchunks + SCAN_BLOCK - 1) / SCAN_BLOCK;
    PC_LAUNCH(K_SD_COLD, sd_cold_count_kernel, dim3(capped(nchunks, SD_GRID_PER_CU)), dim3(256), 0, s, prev, n,
              w.cold, err ? nullptr : w.hdr, gate);
    if (!err) err = w.hdr;
    if (nblocks > 1)
        PC_LAUNCH(K_SD_SCAN, sd_scan_reduce_kernel, dim3((unsigned)nblocks), dim3(SCAN_THREADS), 0, s,
                  (const uint32_t *)w.cold, nchunks, w.part, gate);
    PC_LAUNCH(K_SD_SCAN, sd_scan_apply_kernel, dim3((unsigned)nblocks), dim3(SCAN_THREADS), 0, s,
              (const uint32_t *)w.cold, nchunks, (const uint32_t *)w.part, w.Zc, gate);
    // The MSD levels over next[] in index order (PC_NONE: no element), leaving
    // (t, acc) partitioned by t's 4096-range.
    uint32_t *src_t = nullptr, *src_a = nullptr;
    for (int i = 0; i < p.passes; ++i) {
        uint32_t *dt = (i & 1) ? w.bt : w.at;
        uint32_t *da = (i & 1) ? w.ba : w.aa;
        const int S = p.s[i] + p.k[i];
        const uint64_t ntiles = p.grid[i], nb = p.nbuckets[i], group = seg_group(ntiles);
        const uint64_t cgroups = (ntiles + COUNT_TPW - 1) / COUNT_TPW;
        const unsigned groups = (unsigned)((ntiles + group - 1) / group);
        const unsigned grid = capped(ntiles, SD_GRID_PER_CU), cgrid = capped(cgroups, SD_GRID_PER_CU);
        const uint64_t fixed = (n + DOM_TILE - 1) / DOM_TILE;
        if (i == 0) {
            PC_LAUNCH(K_SD_COUNT, sd_count_kernel<true>, dim3(cgrid), dim3(DOM_THREADS), 0, s, next, n, w.Zc,
                      p.s[i], p.k[i], (const uint32_t *)nullptr, (uint64_t)1, (const uint32_t *)nullptr, w.cnt, w.seg,
                      cgroups, gate);
        } else {
            PC_LAUNCH(K_SD_TILES, sd_tile_map_kernel, dim3((unsigned)nb), dim3(256), 0, s, (const uint32_t *)w.Zc, n,
                      S, nb, w.tfirst, w.tile_bucket, gate);
            PC_LAUNCH(K_SD_COUNT, sd_count_kernel<false>, dim3(cgrid), dim3(DOM_THREADS), 0, s, src_t, n, w.Zc,
                      p.s[i], p.k[i], w.tfirst, nb, w.tile_bucket, w.cnt, w.seg, cgroups, gate);
        }
        const uint32_t *tend = i == 0 ? nullptr : w.tfirst + nb;
        const SegSpace g = seg_space(w, da, groups);
        PC_LAUNCH(K_SD_SEG, sd_seg_reduce_kernel, dim3(groups), dim3(DOM_RADIX), 0, s, w.cnt, w.seg, tend, fixed,
                  group, g.gsum, w.ghas, gate);
        const unsigned carry = groups < CARRY_WAVES_MAX * WAVE ? (groups + WAVE - 1) / WAVE * WAVE : CARRY_WAVES_MAX * WAVE;
        PC_LAUNCH(K_SD_SEG, sd_seg_carry_kernel, dim3(DOM_RADIX), dim3(carry), 0, s, g.gsum, w.ghas, tend, fixed,
                  group, g.gin, gate);
        PC_LAUNCH(K_SD_SEG, sd_seg_scan_kernel, dim3(groups), dim3(DOM_RADIX), 0, s, w.cnt, w.seg, tend, fixed, group,
                  g.gin, w.pre, gate);
        if (i == 0) {
            PC_LAUNCH(K_SD_PASS, sd_dominance_kernel<true>, dim3(grid), dim3(DOM_THREADS), 0, s, next,
                      (const uint32_t *)nullptr, dt, da, n, w.Zc, p.s[i], p.k[i], (const uint32_t *)nullptr,
                      (uint64_t)1, (const uint32_t *)nullptr, w.pre, err, ntiles, gate);
        } else {
            PC_LAUNCH(K_SD_PASS, sd_dominance_kernel<false>, dim3(grid), dim3(DOM_THREADS), 0, s, src_t, src_a, dt,
                      da, n, w.Zc, p.s[i], p.k[i], w.tfirst, nb, w.tile_bucket, w.pre, err, ntiles, gate);
        }
        src_t = dt;
        src_a = da;
    }
    PC_LAUNCH(K_SD_LOCAL, sd_local_kernel, dim3(capped(nchunks, SD_GRID_PER_CU)), dim3(LOC_THREADS), 0, s, src_t, src_a,
              prev, n, w.Zc, dist, gate);
    return PC_OK;
}

// ---- all steps in one launch, for the fallback behind the count over runs --
// The choice between the two is made on the device, and a launch that its gate
// turns off costs about 4.5 us in the stream, so up to SD_PERSISTENT_MAX
// accesses the ten or so steps are the phases of one persistent kernel: a
// phase hands out its chunks from a counter and counts the finished ones, and
// a workgroup goes on once all are finished.  One workgroup per CU: the ends
// of the phases cost about as much as launches then, and less than a tenth of
// what they cost with four (3.0e6 random accesses 0.37 ms, 0.39 as launches,
// 1.14 with four).  Larger calls keep the launches: one workgroup per CU is
// too slow for the tiles (3.0e7: 1.42 against 0.89 ms), and 70 us of gated
// launches are little beside the rest of such a step.  At least 32 workgroups,
// for the carries have 256 chunks however few the tiles are (3000 accesses 70
// us; two workgroups 184, 16 76, 256 104; as launches 89).
constexpr uint64_t SD_PERSISTENT_MAX = 1ull << 22;
constexpr uint64_t SD_WORKGROUPS_MIN = 32;
struct SdJob {
    const uint32_t *prev, *next;
    uint32_t *dist;
    uint64_t n;
    SdPlan p;
    SdWs w;
    uint64_t group[4];
    uint32_t *ctl;        // two zeroed words per phase
    int32_t *status;      // the caller's status word
};
constexpr int SD_PHASES = 3 + 4 * 6 + 1;
static_assert(2 * SD_PHASES <= SD_CTL_WORDS, "two control words per phase");

union SdPersistentLds {
    DomLds dom;
    LocalLds local;
    uint32_t cnt[COUNT_TPW][DOM_RADIX];
};

__global__ __launch_bounds__(DOM_THREADS, 4) void sd_persistent_kernel(SdJob j, const int32_t *gate) {
    static_assert(DOM_THREADS == LOC_THREADS, "one workgroup size for all phases");
    if (gated_off(gate)) return;
    __shared__ SdPersistentLds L;
    __shared__ uint32_t s_tmp[DOM_WAVES], s_has[DOM_WAVES], s_word;
    const uint64_t n = j.n;
    int phase = 0;
    // f(chunk) over [0, chunks), then wait until every workgroup's are done; a
    // workgroup takes a few chunks at a time, since the counter answers one
    // workgroup after the other (about 10 ns each)
    auto run = [&](uint64_t chunks, auto &&f) {
        uint32_t *c = j.ctl + 2 * phase++;
        uint32_t mine = 0;
        uint64_t take = chunks / (4ull * gridDim.x);
        take = take < 1 ? 1 : take > 8 ? 8 : take;
        for (;;) {
            __syncthreads();
            if (threadIdx.x == 0) s_word = atomicAdd(&c[0], (uint32_t)take);
            __syncthreads();
            const uint64_t x = s_word;
            if (x >= chunks) break;
            for (uint64_t y = x; y < x + take && y < chunks; ++y) {
                if (y > x) __syncthreads();
                f(y);
                ++mine;
            }
        }
        finish_phase(&c[1], mine, (uint32_t)chunks, j.status);
    };
    const SdWs &w = j.w;
    const uint64_t nchunks = (n + LOCAL_SPAN - 1) / LOCAL_SPAN, nblocks = (nchunks + SCAN_BLOCK - 1) / SCAN_BLOCK;
    run(nchunks, [&](uint64_t c) { cold_count<DOM_THREADS>(j.prev, n, c, w.cold, s_tmp); });
    run(nblocks, [&](uint64_t c) { scan_reduce(w.cold, nchunks, c, w.part, s_tmp); });
    run(nblocks, [&](uint64_t c) { scan_apply<DOM_THREADS>(w.cold, nchunks, c, w.part, w.Zc, s_tmp); });
    const uint32_t *src_t = j.next, *src_a = nullptr;
#pragma unroll 1
    for (int i = 0; i < j.p.passes; ++i) {
        uint32_t *dt = (i & 1) ? w.bt : w.at, *da = (i & 1) ? w.ba : w.aa;
        const int s = j.p.s[i], k = j.p.k[i];
        const uint64_t nb = j.p.nbuckets[i], group = j.group[i];
        if (i > 0) run(nb, [&](uint64_t c) { map_tiles(w.Zc, n, s + k, nb, c, w.tfirst, w.tile_bucket, s_tmp); });
        else ++phase;
        const uint64_t rows = i > 0 ? (uint64_t)ld_status(&w.tfirst[nb]) : (n + DOM_TILE - 1) / DOM_TILE;
        const uint64_t groups = (rows + group - 1) / group;
        const SegSpace g0 = seg_space(w, da, groups);
        run((rows + COUNT_TPW - 1) / COUNT_TPW, [&](uint64_t c) {
            if (i == 0) count_tiles<true>(src_t, n, w.Zc, s, k, nullptr, 1, nullptr, w.cnt, w.seg, c, L.cnt);
            else count_tiles<false>(src_t, n, w.Zc, s, k, w.tfirst, nb, w.tile_bucket, w.cnt, w.seg, c, L.cnt);
        });
        // (a digit per thread: two groups at a time)
        const int d = (int)threadIdx.x & (DOM_RADIX - 1);
        auto rows_of = [&](uint64_t g, uint64_t *r0, uint64_t *r1) {
            *r0 = g * group;
            *r1 = *r0 + group < rows ? *r0 + group : rows;
            return *r0 < rows;
        };
        run((groups + 1) / 2, [&](uint64_t c) {
            const uint64_t g = 2 * c + threadIdx.x / DOM_RADIX;
            uint64_t r0, r1;
            if (rows_of(g, &r0, &r1)) seg_reduce(w.cnt, w.seg, r0, r1, d, g, g0.gsum, w.ghas);
        });
        run(DOM_RADIX, [&](uint64_t c) { seg_carry(g0.gsum, w.ghas, groups, (int)c, g0.gin, s_tmp, s_has); });
        run((groups + 1) / 2, [&](uint64_t c) {
            const uint64_t g = 2 * c + threadIdx.x / DOM_RADIX;
            uint64_t r0, r1;
            if (rows_of(g, &r0, &r1)) seg_scan(w.cnt, w.seg, r0, r1, d, g, g0.gin, w.pre);
        });
        run(rows, [&](uint64_t c) {
            if (i == 0)
                dominance_tile<true>(L.dom, src_t, nullptr, dt, da, n, w.Zc, s, k, nullptr, 1, nullptr, w.pre,
                                     j.status, c);
            else
                dominance_tile<false>(L.dom, src_t, src_a, dt, da, n, w.Zc, s, k, w.tfirst, nb, w.tile_bucket, w.pre,
                                      j.status, c);
        });
        src_t = dt;
        src_a = da;
    }
    run(nchunks, [&](uint64_t c) { local_range(L.local, src_t, src_a, j.prev, n, w.Zc, j.dist, c); });
}

pc_status stack_distance_rare(const uint32_t *prev, const uint32_t *next, uint64_t n, uint32_t *dist, void *ws,
                              uint32_t *ctl, hipStream_t s, const int32_t *gate, int32_t *status) {
    if (n > SD_PERSISTENT_MAX) return stack_distance_steps(prev, next, n, dist, ws, s, gate, status);
    SdJob j;
    j.prev = prev;
    j.next = next;
    j.dist = dist;
    j.n = n;
    j.p = plan_sd(n);
    j.w = carve_sd(ws, n, j.p);
    for (int i = 0; i < j.p.passes; ++i) j.group[i] = seg_group(j.p.grid[i]);
    j.ctl = ctl;
    j.status = status;
    uint64_t tiles = (n + DOM_TILE - 1) / DOM_TILE;
    if (tiles < SD_WORKGROUPS_MIN) tiles = SD_WORKGROUPS_MIN;
    PC_LAUNCH(K_SD_ALL, sd_persistent_kernel, dim3(capped(tiles, 1)), dim3(DOM_THREADS), 0, s, j, gate);
    return PC_OK;
}

}  // namespace pc

extern "C" {

size_t pc_stack_distance_ws(uint64_t n) {
    const pc::SdPlan p = pc::plan_sd(n);
    return pc::carve_sd(nullptr, n, p).bytes;
}

pc_status pc_stack_distance(const uint32_t *prev, const uint32_t *next, uint64_t n, uint32_t *dist,
                            void *ws, size_t ws_bytes, void *stream) {
    if (n >= (uint64_t)PC_NONE) return PC_ERR_TOO_LARGE;
    if (n > 0 && (!prev || !next || !dist)) return PC_ERR_INVALID;
    if (!ws) return PC_ERR_WORKSPACE;
    if (ws_bytes < pc_stack_distance_ws(n)) return PC_ERR_WORKSPACE;
    return pc::stack_distance_steps(prev, next, n, dist, ws, (hipStream_t)stream, nullptr, nullptr);
}

size_t pc_request_order_ws(void) { return pc::WS_HEADER; }

pc_status pc_request_order(const uint64_t *keys, const uint32_t *depth, const uint64_t *blk_off, uint32_t n_seqs,
                           uint64_t n, uint64_t *keys_out, uint32_t *depth_out, void *ws, size_t ws_bytes,
                           void *stream) {
    if (n >= (uint64_t)PC_NONE) return PC_ERR_TOO_LARGE;
    if (n > 0 && (!keys || !keys_out || !blk_off)) return PC_ERR_INVALID;
    if ((depth == nullptr) != (depth_out == nullptr)) return PC_ERR_INVALID;
    if ((n > 0 && keys == keys_out) || (depth && depth == depth_out)) return PC_ERR_INVALID;
    if (!ws) return PC_ERR_WORKSPACE;
    if (ws_bytes < pc_request_order_ws()) return PC_ERR_WORKSPACE;
    hipStream_t s = (hipStream_t)stream;
    int32_t *hdr = reinterpret_cast<int32_t *>(ws);
    pc_status st = pc::fill_u32(reinterpret_cast<uint32_t *>(hdr), 0u, 1, s);
    if (st != PC_OK || n == 0 || n_seqs == 0) return st;
    const int cus = pc::device_cus();
    uint64_t grid = ((uint64_t)n_seqs + 3) / 4;
    if (grid > (uint64_t)cus * 8) grid = (uint64_t)cus * 8;
    PC_LAUNCH(pc::K_REQ_ORDER, pc::req_order_kernel, dim3((unsigned)grid), dim3(256), 0, s, keys, depth, blk_off,
              n_seqs, n, keys_out, depth_out, hdr);
    return PC_OK;
}

size_t pc_stack_distance_req_ws(void) { return pc::WS_HEADER; }

pc_status pc_stack_distance_req(const uint32_t *prev, const uint32_t *dist, const uint64_t *blk_off, uint32_t n_seqs,
                                uint64_t n, uint32_t *dist_req, void *ws, size_t ws_bytes, void *stream) {
    if (n >= (uint64_t)PC_NONE) return PC_ERR_TOO_LARGE;
    if (n > 0 && (!prev || !dist || !dist_req || !blk_off || n_seqs == 0)) return PC_ERR_INVALID;
    if (n_seqs >= 0x80000000u) return PC_ERR_TOO_LARGE;
    if (!ws) return PC_ERR_WORKSPACE;
    if (ws_bytes < pc_stack_distance_req_ws()) return PC_ERR_WORKSPACE;
    hipStream_t s = (hipStream_t)stream;
    int32_t *hdr = reinterpret_cast<int32_t *>(ws);
    pc_status st = pc::fill_u32(reinterpret_cast<uint32_t *>(hdr), 0u, 1, s);
    if (st != PC_OK || n == 0) return st;
    const int cus = pc::device_cus();
    // Workgroups of one wave where requests are long (they differ in length, and
    // a workgroup's place is free only when all its waves are through), of four
    // and no loads ahead where they are short (1.0e7 accesses in requests of 70:
    // 52 us, 71 the other way).
    const unsigned waves = n / n_seqs >= 256 ? 1 : 4;
    uint64_t grid = ((uint64_t)n_seqs + waves - 1) / waves;
    if (grid > (uint64_t)cus * 256 / waves) grid = (uint64_t)cus * 256 / waves;
    const auto kernel = waves == 1 ? pc::req_dist_kernel<true> : pc::req_dist_kernel<false>;
    PC_LAUNCH(pc::K_REQ_DIST, kernel, dim3((unsigned)grid), dim3(waves * pc::WAVE), 0, s, prev, dist, blk_off, n_seqs,
              n, dist_req, hdr);
    return PC_OK;
}

}  // extern "C"
