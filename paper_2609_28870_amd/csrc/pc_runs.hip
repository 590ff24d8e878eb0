// Exact LRU stack distance from the runs of the prev stream
// (pc_stack_distance_runs).  Same output as pc_stack_distance.
//
// The stack distance of an access is the number of distinct blocks used
// since the previous use of its block (Sec. 5; Appendix B).  With
// v(j) = prev(j) + 1 (0 when cold), #{j < t : v(j) < v(t)} = prev(t) + 1 + D(t),
// so D(t) = Z(t) + C'(t) - prev(t) - 1 with Z(t) the cold accesses before t
// and C'(t) the earlier warm accesses whose previous use is older than t's.
//
// Runs.  Call t a continuation when t - 1 and t are warm and
// prev(t) = prev(t - 1) + 1.  Then the window (prev(t), t) is the window of
// t - 1 without position prev(t) (whose block recurs only at t) and with
// position t - 1 (whose block last occurred at prev(t - 1), outside the new
// window): D(t) = D(t - 1).  A maximal chain of continuations is a run; its
// first access is its head.  Chained block keys make runs long (a request's
// reuse of an earlier request's prefix is one run), about one per request.
//
// Counting over runs.  The previous uses of a run's accesses form the range
// [p, p + len) of positions, p = prev(head); since prev is one-to-one, the
// ranges of different runs are disjoint, so every earlier run lies entirely
// below or above a head's previous use and C'(head of run r) is the sum of
// len(s) over the earlier runs s with p(s) < p(r).  That weighted dominance
// count over the runs is a bottom-up merge by p: at each level an element
// finds its rank in the sibling block by binary search, an element of a
// right block adds the sibling's prefix sum of len at that rank, and the
// merged prefix sums follow from the two blocks' own.
//
// Passes: count heads and cold accesses per 4096-position tile, keeping
// three bits per position (head, cold, last of a run); scan, and decide on the
// device; compact the runs from those bits (head's prev, head position, end
// position, cold count before the head); merge the runs of each block of 2048
// in LDS, then eight blocks a launch; write D from the run list.  prev is
// streamed once.  With more runs than 1/16 of the accesses plus 1024 the
// dominance count of pc_stack_distance runs instead.
#include "pc_internal.h"

namespace pc {

constexpr int RUN_THREADS = 256;
constexpr int RUN_ITEMS = 16;
constexpr int RUN_TILE = RUN_THREADS * RUN_ITEMS;   // 4096 positions
constexpr int RSCAN_THREADS = 1024;
constexpr int RSCAN_TILE = RSCAN_THREADS * 4;

// header words of the runs workspace
constexpr int RW_STATUS = 0;
constexpr int RW_PATH = 1;    // 0 = runs, 1 = pc_stack_distance
constexpr int RW_RUNS = 2;    // number of runs
constexpr int RW_COLD = 3;    // number of cold accesses
constexpr int RW_RUNS_OK = 4; // 1 = the runs path runs (the gate of its kernels)

// the number of runs (written by the scan)
__device__ __forceinline__ uint64_t runs_of(const int32_t *hdr) { return (uint32_t)hdr[RW_RUNS]; }

// This thread's 16 consecutive prev values and the ones just before and
// after them (from the neighbouring lanes, or from memory across waves and
// tiles).
struct RunView {
    uint32_t p[RUN_ITEMS];
    uint32_t before;   // prev(t0 - 1), NONE at t = 0
    uint32_t after;    // prev(t0 + 16), NONE past the end
    uint64_t t0;
};

__device__ __forceinline__ void load_view(const uint32_t *__restrict__ prev, uint64_t n, RunView &v) {
    const uint64_t tile0 = (uint64_t)blockIdx.x * RUN_TILE;
    v.t0 = tile0 + (uint64_t)threadIdx.x * RUN_ITEMS;
    if (v.t0 + RUN_ITEMS <= n && (reinterpret_cast<uintptr_t>(prev) & 15) == 0) {
        const uint4 *q = reinterpret_cast<const uint4 *>(prev + v.t0);
#pragma unroll
        for (int k = 0; k < RUN_ITEMS / 4; ++k) {
            const uint4 x = q[k];
            v.p[4 * k] = x.x;
            v.p[4 * k + 1] = x.y;
            v.p[4 * k + 2] = x.z;
            v.p[4 * k + 3] = x.w;
        }
    } else {
#pragma unroll
        for (int k = 0; k < RUN_ITEMS; ++k) v.p[k] = v.t0 + k < n ? prev[v.t0 + k] : NONE;
    }
    // neighbours inside the wave by DPP, across waves and tiles from memory
    const int lane = threadIdx.x & (WAVE - 1);
    const uint32_t lo = from_lower(v.p[RUN_ITEMS - 1]);
    const uint32_t hi = from_upper(v.p[0]);
    v.before = lane ? lo : (v.t0 > 0 && v.t0 - 1 < n ? prev[v.t0 - 1] : NONE);
    v.after = lane != WAVE - 1 ? hi : (v.t0 + RUN_ITEMS < n ? prev[v.t0 + RUN_ITEMS] : NONE);
    if (v.t0 + RUN_ITEMS > n) v.after = NONE;
}

// warm t that does not continue t - 1's run
__device__ __forceinline__ bool is_head(uint32_t p, uint32_t before) {
    return p != NONE && (before == NONE || p != before + 1);
}

// Per 4096-position tile: the number of run heads and of cold accesses, and
// per thread (16 positions) three bit masks: heads and cold accesses
// (low / high half of .x) and last accesses of runs (.y).
__global__ __launch_bounds__(RUN_THREADS) void runs_count_kernel(const uint32_t *__restrict__ prev, uint64_t n,
                                                                 uint2 *__restrict__ counts,
                                                                 uint2 *__restrict__ marks) {
    __shared__ uint32_t tmp[RUN_THREADS / WAVE];
    RunView v;
    load_view(prev, n, v);
    uint32_t hm = 0, cm = 0, em = 0;
#pragma unroll
    for (int k = 0; k < RUN_ITEMS; ++k) {
        const uint64_t t = v.t0 + k;
        const uint32_t p = v.p[k];
        if (t < n) {
            if (p == NONE) {
                cm |= 1u << k;
            } else {
                if (is_head(p, k ? v.p[k - 1] : v.before)) hm |= 1u << k;
                // last access of its run: the next one is cold, a head, or past the end
                const uint32_t q = k + 1 < RUN_ITEMS ? v.p[k + 1] : v.after;
                if (t + 1 >= n || q == NONE || q != p + 1) em |= 1u << k;
            }
        }
    }
    marks[(uint64_t)blockIdx.x * RUN_THREADS + threadIdx.x] = make_uint2(hm | (cm << 16), em);
    uint32_t th = 0, tc = 0;
    block_excl_scan((uint32_t)__popc(hm), tmp, &th);
    block_excl_scan((uint32_t)__popc(cm), tmp, &tc);
    if (threadIdx.x == 0) counts[blockIdx.x] = make_uint2(th, tc);
}

// Exclusive scan of the per-tile (heads, cold) pairs: sums of RSCAN_TILE
// tiles (only when there are more than that), then every workgroup adds the
// sums before its own and scans its tiles.  Workgroup 0 writes the header,
// the path included: over runs, or the dominance count over accesses when
// there are more runs than the workspace holds (rmax); and clears the control
// words of the latter.
__global__ __launch_bounds__(RSCAN_THREADS) void runs_scan_tiles_kernel(const uint2 *__restrict__ c, uint64_t m,
                                                                        uint2 *__restrict__ tsum) {
    __shared__ uint32_t tmp[RSCAN_THREADS / WAVE];
    const uint64_t t0 = (uint64_t)blockIdx.x * RSCAN_TILE;
    uint32_t a = 0, b = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const uint64_t i = t0 + (uint64_t)k * RSCAN_THREADS + threadIdx.x;
        if (i < m) {
            a += c[i].x;
            b += c[i].y;
        }
    }
    uint32_t ta = 0, tb = 0;
    block_excl_scan(a, tmp, &ta);
    block_excl_scan(b, tmp, &tb);
    if (threadIdx.x == 0) tsum[blockIdx.x] = make_uint2(ta, tb);
}

__global__ __launch_bounds__(RSCAN_THREADS) void runs_scan_kernel(const uint2 *__restrict__ c, uint64_t m,
                                                                  const uint2 *__restrict__ tsum,
                                                                  uint2 *__restrict__ out, uint64_t rmax,
                                                                  int32_t *__restrict__ hdr, uint32_t *__restrict__ ctl,
                                                                  uint32_t ctl_words) {
    __shared__ uint32_t tmp[RSCAN_THREADS / WAVE];
    uint32_t ma = 0, mb = 0, aa = 0, ab = 0;   // before this workgroup, and in all
    if (gridDim.x > 1) {
        for (uint32_t i = threadIdx.x; i < gridDim.x; i += RSCAN_THREADS) {
            const uint2 v = tsum[i];
            aa += v.x;
            ab += v.y;
            ma += i < blockIdx.x ? v.x : 0u;
            mb += i < blockIdx.x ? v.y : 0u;
        }
    }
    uint32_t ba = 0, bb = 0, runs = 0, cold = 0;
    block_excl_scan(ma, tmp, &ba);
    block_excl_scan(mb, tmp, &bb);
    block_excl_scan(aa, tmp, &runs);
    block_excl_scan(ab, tmp, &cold);
    const uint64_t i0 = (uint64_t)blockIdx.x * RSCAN_TILE + (uint64_t)threadIdx.x * 4;
    uint2 v[4];
    uint32_t a = 0, b = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        v[k] = i0 + k < m ? c[i0 + k] : make_uint2(0u, 0u);
        a += v[k].x;
        b += v[k].y;
    }
    uint32_t ta = 0, tb = 0;
    uint32_t ra = ba + block_excl_scan(a, tmp, &ta);
    uint32_t rb = bb + block_excl_scan(b, tmp, &tb);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        if (i0 + k < m) out[i0 + k] = make_uint2(ra, rb);
        ra += v[k].x;
        rb += v[k].y;
    }
    if (blockIdx.x != 0) return;
    if (gridDim.x == 1) {
        runs = ta;
        cold = tb;
    }
    if (threadIdx.x == 0) {
        const bool over = runs > rmax;
        hdr[RW_STATUS] = 0;
        hdr[RW_PATH] = over ? 1 : 0;
        hdr[RW_RUNS] = (int32_t)runs;
        hdr[RW_COLD] = (int32_t)cold;
        hdr[RW_RUNS_OK] = over ? 0 : 1;
    }
    for (uint32_t i = threadIdx.x; i < ctl_words; i += RSCAN_THREADS) ctl[i] = 0;
}

// Per run s (in time order): p[s] = prev(head), h[s] = head position,
// e[s] = last position, z[s] = cold accesses before the head; from the
// count pass's bit masks, reading prev only at the heads.
__global__ __launch_bounds__(RUN_THREADS) void runs_compact_kernel(const uint32_t *__restrict__ prev, uint64_t n,
                                                                   const uint2 *__restrict__ off,
                                                                   const uint2 *__restrict__ marks,
                                                                   uint32_t *__restrict__ rp, uint32_t *__restrict__ rh,
                                                                   uint32_t *__restrict__ re,
                                                                   uint32_t *__restrict__ rz, uint64_t tiles,
                                                                   const int32_t *__restrict__ hdr) {
    if (!hdr[RW_RUNS_OK]) return;
    __shared__ uint32_t tmp[RUN_THREADS / WAVE];
    for (uint64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const uint64_t t0 = tile * RUN_TILE + (uint64_t)threadIdx.x * RUN_ITEMS;
        const uint2 mk = marks[tile * RUN_THREADS + threadIdx.x];
        const uint32_t hm = mk.x & 0xFFFFu, cm = mk.x >> 16, em = mk.y;
        uint32_t th = 0, tc = 0;
        const uint2 o = off[tile];
        const uint32_t hs0 = o.x + block_excl_scan((uint32_t)__popc(hm), tmp, &th);   // runs started before t0
        const uint32_t cs0 = o.y + block_excl_scan((uint32_t)__popc(cm), tmp, &tc);
        // heads: one per set bit, numbered in position order
        for (uint32_t m = hm; m; m &= m - 1) {
            const int k = __builtin_ctz(m);
            const uint32_t below = (1u << k) - 1;
            const uint32_t s = hs0 + (uint32_t)__popc(hm & below);
            rp[s] = prev[t0 + k];
            rh[s] = (uint32_t)(t0 + k);
            rz[s] = cs0 + (uint32_t)__popc(cm & below);
        }
        // run ends: the run is the last one started at or before the position
        for (uint32_t m = em; m; m &= m - 1) {
            const int k = __builtin_ctz(m);
            const uint32_t upto = (k == 31) ? ~0u : (2u << k) - 1;
            re[hs0 + (uint32_t)__popc(hm & upto) - 1] = (uint32_t)(t0 + k);
        }
    }
}

// The first levels of the merge: each workgroup sorts BLOCK_RUNS consecutive
// runs by p in LDS, bottom up, with the inclusive prefix sums of their lengths
// and each run's sum over the earlier runs of the block with a smaller p.  The
// p are distinct when prev is one-to-one; runs with equal p (any other prev)
// keep their order, here and in the later merges, so that each run gets a place
// of its own and no index is read from a place that was never written.
constexpr int BLOCK_THREADS = 1024;
constexpr int BLOCK_ITEMS = 2;
constexpr int BLOCK_RUNS = BLOCK_THREADS * BLOCK_ITEMS;
constexpr int BLOCK_LEVELS = 11;
static_assert(BLOCK_RUNS == 1 << BLOCK_LEVELS, "a block is a whole number of levels");
__global__ __launch_bounds__(BLOCK_THREADS) void runs_block_kernel(
    const uint32_t *__restrict__ rp, const uint32_t *__restrict__ rh, const uint32_t *__restrict__ re,
    uint32_t *__restrict__ key, uint32_t *__restrict__ pre, uint32_t *__restrict__ idx, uint32_t *__restrict__ acc,
    const int32_t *__restrict__ hdr) {
    if (!hdr[RW_RUNS_OK]) return;
    __shared__ uint32_t s_key[2][BLOCK_RUNS], s_pre[2][BLOCK_RUNS], s_acc[BLOCK_RUNS];
    __shared__ uint16_t s_idx[2][BLOCK_RUNS];
    const uint64_t r = runs_of(hdr);
    for (uint64_t b0 = (uint64_t)blockIdx.x * BLOCK_RUNS; b0 < r; b0 += (uint64_t)gridDim.x * BLOCK_RUNS) {
        const int m = r - b0 < (uint64_t)BLOCK_RUNS ? (int)(r - b0) : BLOCK_RUNS;
        for (int i = threadIdx.x; i < m; i += BLOCK_THREADS) {
            s_key[0][i] = rp[b0 + i];
            s_pre[0][i] = re[b0 + i] - rh[b0 + i] + 1;
            s_idx[0][i] = (uint16_t)i;
            s_acc[i] = 0;
        }
        int cur = 0;
        for (int lvl = 0; (1 << lvl) < m; ++lvl) {
            __syncthreads();
#pragma unroll
            for (int q = 0; q < BLOCK_ITEMS; ++q) {
                const int i = (int)threadIdx.x + q * BLOCK_THREADS;
                if (i >= m) continue;
                const int blk = i >> lvl, sb = (blk ^ 1) << lvl;
                int lo = sb < m ? sb : m, hi = sb + (1 << lvl) < m ? sb + (1 << lvl) : m;
                const int first = lo;
                const uint32_t k = s_key[cur][i], from = k + (uint32_t)(blk & 1);
                while (lo < hi) {   // the sibling's keys before k
                    const int mid = (lo + hi) >> 1;
                    if (s_key[cur][mid] < from) lo = mid + 1;
                    else hi = mid;
                }
                const int rank = lo - first;
                const uint32_t below = rank ? s_pre[cur][lo - 1] : 0u;   // sibling weights with smaller keys
                const int id = s_idx[cur][i];
                if (blk & 1) s_acc[id] += below;                          // the sibling holds the earlier runs
                const int at = ((blk >> 1) << (lvl + 1)) + (i - (blk << lvl)) + rank;
                s_key[cur ^ 1][at] = k;
                s_pre[cur ^ 1][at] = s_pre[cur][i] + below;
                s_idx[cur ^ 1][at] = (uint16_t)id;
            }
            cur ^= 1;
        }
        __syncthreads();
        for (int i = threadIdx.x; i < m; i += BLOCK_THREADS) {
            key[b0 + i] = s_key[cur][i];
            pre[b0 + i] = s_pre[cur][i];
            idx[b0 + i] = (uint32_t)b0 + s_idx[cur][i];
            acc[b0 + i] = s_acc[i];
        }
        __syncthreads();   // the block has left the LDS before the next one comes in
    }
}

// Three more levels a launch: groups of MERGE_WAYS blocks of 2^lvl runs sorted
// by p become blocks of 2^(lvl+3).  A run finds its rank in each of its seven
// sibling blocks (the binary searches advance together, so a step costs one
// memory latency for all of them): the earlier siblings' sums below it are
// added to its count, all siblings' ranks and sums place it in the merged
// block.
constexpr int MERGE_BITS = 3;
constexpr int MERGE_WAYS = 1 << MERGE_BITS;
__global__ __launch_bounds__(256) void runs_merge_kernel(const uint32_t *__restrict__ key, const uint32_t *__restrict__ pre,
                                                         const uint32_t *__restrict__ idx, int lvl,
                                                         uint32_t *__restrict__ key2, uint32_t *__restrict__ pre2,
                                                         uint32_t *__restrict__ idx2, uint32_t *__restrict__ acc,
                                                         const int32_t *__restrict__ hdr) {
    if (!hdr[RW_RUNS_OK]) return;
    const uint64_t r = runs_of(hdr);
    if ((1ull << lvl) >= r) return;   // the merge took fewer levels
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < r; i += (uint64_t)gridDim.x * blockDim.x) {
        const uint64_t blk = i >> lvl, g0 = (blk >> MERGE_BITS) << (lvl + MERGE_BITS);
        const int mine = (int)(blk & (MERGE_WAYS - 1));
        const uint32_t k = key[i];
        // (positions fit 32 bits: r is at most n / 16 + 1024)
        uint32_t lo[MERGE_WAYS], hi[MERGE_WAYS];
#pragma unroll
        for (int x = 0; x < MERGE_WAYS; ++x) {
            const uint64_t a = g0 + ((uint64_t)x << lvl), e = a + (1ull << lvl);
            lo[x] = (uint32_t)(a < r ? a : r);
            hi[x] = x == mine ? lo[x] : (uint32_t)(e < r ? e : r);   // its own block: no search
        }
        for (int step = 0; step <= lvl; ++step) {
            uint32_t v[MERGE_WAYS];
#pragma unroll
            for (int x = 0; x < MERGE_WAYS; ++x) v[x] = lo[x] < hi[x] ? key[(lo[x] + hi[x]) >> 1] : 0u;
#pragma unroll
            for (int x = 0; x < MERGE_WAYS; ++x) {
                const uint32_t mid = (lo[x] + hi[x]) >> 1;
                if (lo[x] < hi[x]) {
                    if (v[x] < k + (x < mine ? 1u : 0u)) lo[x] = mid + 1;
                    else hi[x] = mid;
                }
            }
        }
        uint32_t earlier = 0, below = 0;
        uint64_t rank = 0;
#pragma unroll
        for (int x = 0; x < MERGE_WAYS; ++x) {
            const uint64_t a = g0 + ((uint64_t)x << lvl);
            const uint32_t first = (uint32_t)(a < r ? a : r);
            const uint32_t w = lo[x] > first ? pre[lo[x] - 1] : 0u;   // (zero for its own block)
            rank += lo[x] - first;
            below += w;
            if (x < mine) earlier += w;
        }
        const uint32_t id = idx[i];
        if (earlier) acc[id] += earlier;
        const uint64_t q = g0 + (i - (blk << lvl)) + rank;
        key2[q] = k;
        pre2[q] = pre[i] + below;
        idx2[q] = id;
    }
}

// D of every position from the run list alone: a warm position lies in
// exactly one run [h, e], every other position is cold.  The runs that can
// touch a tile are the one in progress at its start and those starting in
// it; a thread finds the run at its first position by binary search and
// walks on.  A run's distance is z + acc - p - 1.  Bound: the stores (8.0e8
// accesses 0.586 ms, 5.5 TB/s; with the search and the run's words read from
// memory as needed, a chain of five loads a tile, 0.765).
__global__ __launch_bounds__(RUN_THREADS) void runs_fill_kernel(uint64_t n, const uint2 *__restrict__ off,
                                                                uint64_t tiles, const uint32_t *__restrict__ rh,
                                                                const uint32_t *__restrict__ re,
                                                                const uint32_t *__restrict__ rp,
                                                                const uint32_t *__restrict__ rz,
                                                                const uint32_t *__restrict__ acc,
                                                                uint32_t *__restrict__ dist,
                                                                const int32_t *__restrict__ hdr) {
    if (!hdr[RW_RUNS_OK]) return;
    const uint64_t r = runs_of(hdr);
    const int tid = threadIdx.x;
    // The runs that a tile's positions may lie in are [lo, hi): the ones that
    // start in it and the last one before.  Mostly they are few; then their
    // heads, ends and distances pass through LDS, one per thread, loaded while
    // the tile before is written (and the tile's bounds while the one before
    // that is).
    __shared__ uint32_t s_head[2][RUN_THREADS], s_end[2][RUN_THREADS], s_dist[2][RUN_THREADS];
    struct Bounds {
        uint32_t lo, hi;
    };
    auto bounds = [&](uint64_t tile) {
        Bounds b{0u, 0u};
        if (tile < tiles) {
            const uint32_t first = off[tile].x;
            b.lo = first ? first - 1 : 0u;
            b.hi = tile + 1 < tiles ? off[tile + 1].x : (uint32_t)r;
        }
        return b;
    };
    uint32_t h = 0, e = 0, z = 0, c = 0, p = 0;
    auto fetch = [&](const Bounds &b) {
        if ((uint32_t)tid < b.hi - b.lo && b.hi - b.lo <= RUN_THREADS) {
            const uint32_t k = b.lo + (uint32_t)tid;
            h = rh[k];
            e = re[k];
            z = rz[k];
            c = acc[k];
            p = rp[k];
        }
    };
    Bounds now = bounds(blockIdx.x), next = bounds((uint64_t)blockIdx.x + gridDim.x);
    fetch(now);
    int buf = 0;
    const bool vec = (reinterpret_cast<uintptr_t>(dist) & 15) == 0;
    // thread i holds positions tile0 + 1024 g + 4 i .. + 3 for g = 0..3
    // (increasing), so each 16-byte store covers 1 KB across the wave
    auto write = [&](uint64_t tile, uint32_t runs, auto head_of, auto end_of, auto dist_of) {
        const uint64_t t0 = tile * RUN_TILE + (uint64_t)tid * 4;
        // the runs with head <= t0
        uint32_t lo = 0, hi = runs;
        while (lo < hi) {
            const uint32_t m = (lo + hi) >> 1;
            if (head_of(m) <= t0) lo = m + 1;
            else hi = m;
        }
        uint32_t s = lo;   // the current run is s - 1, the next one s
        // the current run's end and distance and the next run's head, in
        // registers: read only where a run starts
        bool in_run = s > 0;
        uint64_t end = in_run ? end_of(s - 1) : 0;
        uint32_t dv = in_run ? dist_of(s - 1) : NONE;
        uint64_t next_head = s < runs ? head_of(s) : ~0ull;
#pragma unroll
        for (int g = 0; g < RUN_ITEMS / 4; ++g) {
            const uint64_t tg = t0 + (uint64_t)g * (RUN_THREADS * 4);
            uint32_t d[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const uint64_t t = tg + k;
                while (t >= next_head) {
                    in_run = true;
                    end = end_of(s);
                    dv = dist_of(s);
                    ++s;
                    next_head = s < runs ? head_of(s) : ~0ull;
                }
                d[k] = (in_run && end >= t) ? dv : NONE;
            }
            if (vec && tg + 4 <= n) {
                *reinterpret_cast<uint4 *>(dist + tg) = make_uint4(d[0], d[1], d[2], d[3]);
            } else {
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if (tg + k < n) dist[tg + k] = d[k];
            }
        }
    };
    for (uint64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x, buf ^= 1) {
        const uint32_t runs = now.hi - now.lo;
        if (runs <= RUN_THREADS && (uint32_t)tid < runs) {
            s_head[buf][tid] = h;
            s_end[buf][tid] = e;
            s_dist[buf][tid] = z + c - p - 1;
        }
        __syncthreads();
        fetch(next);
        const Bounds after = bounds(tile + 2 * (uint64_t)gridDim.x);
        if (runs <= RUN_THREADS)
            write(
                tile, runs, [&](uint32_t k) -> uint64_t { return s_head[buf][k]; },
                [&](uint32_t k) -> uint64_t { return s_end[buf][k]; }, [&](uint32_t k) { return s_dist[buf][k]; });
        else
            write(
                tile, runs, [&](uint32_t k) -> uint64_t { return rh[now.lo + k]; },
                [&](uint32_t k) -> uint64_t { return re[now.lo + k]; },
                [&](uint32_t k) { return rz[now.lo + k] + acc[now.lo + k] - rp[now.lo + k] - 1; });
        now = next;
        next = after;
    }
}

static uint64_t runs_max(uint64_t n) { return n / 16 + 1024; }

struct RunsWs {
    int32_t *hdr;
    uint32_t *ctl;   // control words of the fallback
    void *sd;   // pc_stack_distance workspace (the fallback); the arrays below live inside it
    size_t sd_bytes;
    uint2 *counts, *tsum, *off, *marks;
    uint32_t *rp, *rh, *re, *rz, *acc, *key[2], *pre[2], *idx[2];
    size_t bytes;
};

static RunsWs carve_runs(void *ws, uint64_t n) {
    Carver c{(char *)ws, 0};
    RunsWs w;
    w.hdr = c.take<int32_t>(WS_HEADER / sizeof(int32_t));
    w.ctl = c.take<uint32_t>(SD_CTL_WORDS);
    w.sd_bytes = pc_stack_distance_ws(n);
    const size_t sd_at = c.off;
    const uint64_t tiles = (n + RUN_TILE - 1) / RUN_TILE;
    const uint64_t rm = runs_max(n);
    w.counts = c.take<uint2>(tiles);
    w.tsum = c.take<uint2>((tiles + RSCAN_TILE - 1) / RSCAN_TILE + 1);
    w.off = c.take<uint2>(tiles);
    w.marks = c.take<uint2>(tiles * RUN_THREADS);
    w.rp = c.take<uint32_t>(rm);
    w.rh = c.take<uint32_t>(rm);
    w.re = c.take<uint32_t>(rm);
    w.rz = c.take<uint32_t>(rm);
    w.acc = c.take<uint32_t>(rm);
    for (int i = 0; i < 2; ++i) {
        w.key[i] = c.take<uint32_t>(rm);
        w.pre[i] = c.take<uint32_t>(rm);
        w.idx[i] = c.take<uint32_t>(rm);
    }
    w.sd = ws ? (char *)ws + sd_at : nullptr;
    const size_t own = c.off;
    w.bytes = own > sd_at + w.sd_bytes ? own : sd_at + w.sd_bytes;
    return w;
}

}  // namespace pc

extern "C" {

size_t pc_stack_distance_runs_ws(uint64_t n) { return pc::carve_runs(nullptr, n).bytes; }

pc_status pc_stack_distance_runs(const uint32_t *prev, const uint32_t *next, uint64_t n, uint32_t *dist, void *ws,
                                 size_t ws_bytes, void *stream) {
    using namespace pc;
    if (n >= (uint64_t)PC_NONE) return PC_ERR_TOO_LARGE;
    if (n > 0 && (!prev || !next || !dist)) return PC_ERR_INVALID;
    if (!ws) return PC_ERR_WORKSPACE;
    if (ws_bytes < pc_stack_distance_runs_ws(n)) return PC_ERR_WORKSPACE;
    hipStream_t s = (hipStream_t)stream;
    const RunsWs w = carve_runs(ws, n);
    if (n == 0) return fill_u32(reinterpret_cast<uint32_t *>(w.hdr), 0u, 8, s);
    pc_status st;
    const uint64_t tiles = (n + RUN_TILE - 1) / RUN_TILE;
    const uint64_t stiles = (tiles + RSCAN_TILE - 1) / RSCAN_TILE;
    const uint64_t rm = runs_max(n);
    PC_LAUNCH(K_RUNS_COUNT, runs_count_kernel, dim3((unsigned)tiles), dim3(RUN_THREADS), 0, s, prev, n, w.counts,
              w.marks);
    if (stiles > 1)
        PC_LAUNCH(K_RUNS_SCAN, runs_scan_tiles_kernel, dim3((unsigned)stiles), dim3(RSCAN_THREADS), 0, s,
                  (const uint2 *)w.counts, tiles, w.tsum);
    // the path is decided on the device, so nothing here waits for the GPU:
    // every later launch is gated on the decision, and the launches of the
    // path not taken return at once (grids capped per compute unit)
    PC_LAUNCH(K_RUNS_SCAN, runs_scan_kernel, dim3((unsigned)stiles), dim3(RSCAN_THREADS), 0, s,
              (const uint2 *)w.counts, tiles, (const uint2 *)w.tsum, w.off, rm, w.hdr, w.ctl, (uint32_t)SD_CTL_WORDS);
    if ((st = stack_distance_rare(prev, next, n, dist, w.sd, w.ctl, s, w.hdr + RW_PATH, w.hdr + RW_STATUS)) != PC_OK)
        return st;
    const int32_t *ok = w.hdr;
    PC_LAUNCH(K_RUNS_COMPACT, runs_compact_kernel, dim3(capped(tiles, 16)), dim3(RUN_THREADS), 0, s, prev, n,
              (const uint2 *)w.off, (const uint2 *)w.marks, w.rp, w.rh, w.re, w.rz, tiles, ok);
    PC_LAUNCH(K_RUNS_MERGE, runs_block_kernel, dim3(capped((rm + BLOCK_RUNS - 1) / BLOCK_RUNS, 4)),
              dim3(BLOCK_THREADS), 0, s, (const uint32_t *)w.rp, (const uint32_t *)w.rh, (const uint32_t *)w.re,
              w.key[0], w.pre[0], w.idx[0], w.acc, ok);
    // one launch per three levels the largest run count needs; the levels past
    // the actual count return at once
    const unsigned rg = capped((rm + 255) / 256, 16);
    int cur = 0;
    for (int lvl = BLOCK_LEVELS; (1ull << lvl) < rm; lvl += MERGE_BITS) {
        PC_LAUNCH(K_RUNS_MERGE, runs_merge_kernel, dim3(rg), dim3(256), 0, s, (const uint32_t *)w.key[cur],
                  (const uint32_t *)w.pre[cur], (const uint32_t *)w.idx[cur], lvl, w.key[cur ^ 1], w.pre[cur ^ 1],
                  w.idx[cur ^ 1], w.acc, ok);
        cur ^= 1;
    }
    PC_LAUNCH(K_RUNS_FILL, runs_fill_kernel, dim3(capped(tiles, 32)), dim3(RUN_THREADS), 0, s, n,
              (const uint2 *)w.off, tiles, (const uint32_t *)w.rh, (const uint32_t *)w.re, (const uint32_t *)w.rp,
              (const uint32_t *)w.rz, (const uint32_t *)w.acc, dist, ok);
    return PC_OK;
}

}  // extern "C"
