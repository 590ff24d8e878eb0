// Previous / next use of every access (pc_prev_next_use).
//
// prev[t] = last earlier position with the same key, next[t] = first later
// one.  The paper's offline analysis ranks blocks by time until next access
// (Sec. 3.2 Belady; Sec. 5.2 BeladyCompute); prev == none marks a compulsory
// miss (Sec. 4.6).
//
// GPU mapping: a stable LSD radix sort of (key, t) groups equal keys with t
// ascending; neighbours in sorted order are exactly the (prev, next) links.
// Keys are 64-bit hashes, so sorting by their low 32 bits already makes
// equal keys contiguous except where different keys share those bits; the
// link step resolves such short "mixed" runs by scanning them, and when a
// run is too long to scan it flags the four passes over the high bits and a
// second link, one persistent launch (then the full 64-bit sort makes equal
// keys adjacent).
//   * the four 8-bit digit histograms of a group of passes come from the
//     caller (the hash kernel counts them while it writes the keys) or from
//     one counting pass (LDS-privatised, then global atomics), whose last
//     workgroup scans them into digit bases;
//   * each of the four sort passes is a single "onesweep" kernel: a
//     workgroup takes the next tile from an atomic counter (so every tile it
//     waits on is already running), ranks its elements (8192, fewer in small
//     calls) by digit with wave ballots (stable: lanes in order, waves in
//     order), publishes its per-digit counts and reads its predecessors' with
//     a decoupled look-back, then writes the tile out through LDS so each digit run is a
//     contiguous burst;
//   * the link + partition kernels read sorted neighbours into (t, prev,
//     next) triples and move them back to time order (see below).
// Waits in the look-back are bounded: after the spin limit the kernel
// records an error in the workspace header instead of hanging.
//
// Inside the library the same kernels also serve a count the GPU wrote
// (n_dev: the chained prev/next sorts the accesses it left unresolved, a
// number it only knows on the device): grids are sized for the host bound n,
// workgroups past the device count return at once, and every launch can be
// gated on a device word, so no call ever waits for the GPU.
#include "pc_internal.h"

namespace pc {

constexpr int RADIX = 256;
constexpr int SORT_THREADS = 512;
constexpr int SORT_WAVES = SORT_THREADS / WAVE;
constexpr int SORT_ITEMS = 16;
constexpr int SORT_TILE = SORT_THREADS * SORT_ITEMS;   // 8192
// Small calls take small tiles: with few tiles a pass is one tile's latency.
// us per pass with tiles of 2048 / 4096 / 8192 keys, launch included: 1400 to
// 6000 keys 8.8 10.2 13.0, 4.5e4 11.1 11.1 13.0, 4.5e5 18.9 18.6 19.4, 1.0e6
// 26 20 21 (the runs of a tile's digits in the output get short).
constexpr uint64_t SORT_MAX_4 = 1u << 18, SORT_MAX_8 = 1u << 20;
constexpr int SORT_PASSES = 8;
constexpr uint64_t FLAG_AGG = 1ull << 32;
constexpr uint64_t FLAG_INC = 1ull << 33;
constexpr uint32_t SPIN_LIMIT = 1u << 22;
constexpr int LOOKBACK = 4;   // tiles per look-back step (33.5 M keys: 223 us a pass, one at a time 229, 8 228)

// Words of the control block (zeroed before each call): tile counters of the
// passes, tickets, and for the persistent kernel a chunk counter and a count
// of finished chunks per phase.
enum CtlWord {
    CTL_TILE = 0,          // + pass: next tile of a sort pass
    CTL_TICKET = 8,        // blocks of the histogram kernel that are through
    CTL_PHASE = 16,        // + 2 * phase: next chunk, finished chunks
    CTL_WORDS = 48
};
constexpr int HIST_DIGITS = SORT_PASSES / 2;
// The counting pass: eight loads in flight per thread, one workgroup per CU (each
// adds its 1024 bins to the same words at the end; 3.4e7 keys 58 us, one load at
// a time in four workgroups of 256 threads 93; a step of 4.5e5 and 2.4e6 keys 30 and 51).
constexpr int HIST_THREADS = 512, HIST_AHEAD = 8;

// Histogram of HIST_DIGITS byte digits from p0 on over keys[lo, hi), LDS to
// global (all threads of the workgroup; h: HIST_DIGITS * RADIX words of LDS)
__device__ __forceinline__ void digit_hist(const uint64_t *keys, uint64_t lo, uint64_t hi, uint64_t stride, int p0,
                                           uint32_t *h, uint32_t *hist) {
    for (int i = threadIdx.x; i < HIST_DIGITS * RADIX; i += blockDim.x) h[i] = 0;
    __syncthreads();
    auto count = [&](uint64_t key) {
        const uint32_t k = (uint32_t)(key >> (8 * p0));
#pragma unroll
        for (int p = 0; p < HIST_DIGITS; ++p) atomicAdd(&h[p * RADIX + ((k >> (8 * p)) & 0xFF)], 1u);
    };
    // HIST_AHEAD loads in flight per thread
    uint64_t i = lo + threadIdx.x;
    for (; i + (HIST_AHEAD - 1) * stride < hi; i += HIST_AHEAD * stride) {
        uint64_t k[HIST_AHEAD];
#pragma unroll
        for (int q = 0; q < HIST_AHEAD; ++q) k[q] = keys[i + q * stride];
#pragma unroll
        for (int q = 0; q < HIST_AHEAD; ++q) count(k[q]);
    }
    for (; i < hi; i += stride) count(keys[i]);
    __syncthreads();
    for (int i = threadIdx.x; i < HIST_DIGITS * RADIX; i += blockDim.x)
        if (h[i]) atomicAdd(&hist[p0 * RADIX + i], h[i]);
}

// Exclusive scan of each of HIST_DIGITS 256-bin rows -> digit bases (one
// workgroup of at least 256 threads); a row that does not sum to n (a
// histogram handed in by the caller) is reported
__device__ __forceinline__ void digit_starts(const uint32_t *rows, uint32_t *start, uint64_t n, uint32_t *tmp,
                                             int32_t *err) {
    for (int p = 0; p < HIST_DIGITS; ++p) {
        uint32_t total;
        const bool in = (int)threadIdx.x < RADIX;
        const uint32_t v = in ? ld_status(&rows[p * RADIX + threadIdx.x]) : 0u;
        const uint32_t e = block_excl_scan(v, tmp, &total);
        if (in) start[p * RADIX + threadIdx.x] = e;
        if (threadIdx.x == 0 && (uint64_t)total != n) atomicOr(err, DEV_ERR_BAD_HIST);
    }
}

// First launch of a call: clears the control block, the histograms, the
// partition cursors and the look-back status, and, with the low bytes'
// histograms handed in, turns them into digit starts.
__global__ __launch_bounds__(256) void sort_init_kernel(Fills f, const uint32_t *__restrict__ key_hist,
                                                        uint32_t *__restrict__ start, uint64_t n,
                                                        int32_t *__restrict__ err, const uint32_t *__restrict__ n_dev,
                                                        const int32_t *__restrict__ gate) {
    if (gated_off(gate)) return;
    __shared__ uint32_t tmp[256 / WAVE];
    fill_segments(f);
    if (key_hist && blockIdx.x == 0) digit_starts(key_hist, start, dev_count(n, n_dev), tmp, err);
}

// Histograms of the four low byte digits in one read of the keys; the last
// block to finish turns them into digit starts.
__global__ __launch_bounds__(HIST_THREADS) void sort_hist_kernel(
    const uint64_t *__restrict__ keys, uint64_t n, uint32_t *hist, uint32_t *__restrict__ start,
    uint32_t *__restrict__ ctl, int32_t *__restrict__ err, const uint32_t *__restrict__ n_dev,
    const int32_t *__restrict__ gate) {
    if (gated_off(gate)) return;
    n = dev_count(n, n_dev);
    __shared__ uint32_t h[HIST_DIGITS * RADIX];
    __shared__ uint32_t tmp[HIST_THREADS / WAVE];
    __shared__ uint32_t ticket;
    digit_hist(keys, (uint64_t)blockIdx.x * blockDim.x, n, (uint64_t)gridDim.x * blockDim.x, 0, h, hist);
    atomics_performed();
    __syncthreads();
    if (threadIdx.x == 0) ticket = atomicAdd(&ctl[CTL_TICKET], 1u);
    __syncthreads();
    if (ticket == gridDim.x - 1) digit_starts(hist, start, n, tmp, err);
}

// Large tiles make each digit's run in the output long (about 32 elements
// of 8192), so the scattered writes are mostly whole lines; the tile is
// staged twice through one buffer (keys, then values) and the per-wave digit
// counters are 16-bit (a tile holds at most 8192 elements), which keeps two
// workgroups on a CU
template <int ITEMS>
struct SortLds {
    uint64_t stage[ITEMS * SORT_THREADS];
    uint16_t wcnt[SORT_WAVES][RADIX];
    uint32_t lstart[RADIX];
    uint32_t gbase[RADIX];
    uint32_t tmp[SORT_WAVES];
    uint32_t tile;
};

// One tile of a pass: the workgroup takes the next tile from the counter
// (tiles are handed out in order, so every tile a look-back waits on belongs
// to a workgroup already running it); false when none is left.
template <int ITEMS>
__device__ __forceinline__ bool sort_tile(SortLds<ITEMS> &L, const uint64_t *keys_in, const uint32_t *vals_in,
                                          uint64_t *keys_out, uint32_t *vals_out, uint64_t n, int shift,
                                          const uint32_t *start, uint64_t *status, uint32_t *counter, uint32_t epoch,
                                          int32_t *err) {
    constexpr int TILE = ITEMS * SORT_THREADS;
    // (an opaque copy: in a loop over tiles what is derived from it is worked
    // out per tile instead of being held, and spilled, across the loop)
    int tid = threadIdx.x;
    __asm__ volatile("" : "+v"(tid));
    const int lane = tid & (WAVE - 1);
    const int w = tid / WAVE;
    if (tid == 0) L.tile = atomicAdd(counter, 1u);
    for (int i = tid; i < SORT_WAVES * RADIX / 2; i += SORT_THREADS) reinterpret_cast<uint32_t *>(&L.wcnt[0][0])[i] = 0;
    __syncthreads();
    const uint32_t tile = L.tile;
    const uint64_t base = (uint64_t)tile * TILE;
    if (base >= n) return false;

    uint64_t k[ITEMS];
    uint32_t v[ITEMS];
    uint32_t pos[ITEMS];
    bool ok[ITEMS];
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        const uint64_t idx = base + (uint64_t)(w * ITEMS + j) * WAVE + lane;
        ok[j] = idx < n;
        k[j] = ok[j] ? keys_in[idx] : 0ull;
        v[j] = ok[j] ? (vals_in ? vals_in[idx] : (uint32_t)idx) : 0u;
    }
    // stable rank inside the wave: lanes with the same digit are matched by
    // eight ballots; a per-wave running count orders the wave's chunks
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        const uint32_t d = (uint32_t)(k[j] >> shift) & 0xFF;
        const uint64_t m = match_digit<8>(d, ballot(ok[j]));
        const uint32_t before = mbcnt(m);
        uint32_t cur = 0;
        if (ok[j]) cur = L.wcnt[w][d];
        pos[j] = cur + before;
        if (ok[j] && before == 0) L.wcnt[w][d] = (uint16_t)(cur + (uint32_t)__popcll(m));
    }
    __syncthreads();
    uint32_t cnt = 0;
    if (tid < RADIX) {
        for (int x = 0; x < SORT_WAVES; ++x) {
            const uint32_t c = L.wcnt[x][tid];
            L.wcnt[x][tid] = (uint16_t)cnt;
            cnt += c;
        }
    }
    uint32_t total;
    const uint32_t lst = block_excl_scan(tid < RADIX ? cnt : 0u, L.tmp, &total);
    if (tid < RADIX) L.lstart[tid] = lst;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        if (ok[j]) {
            const uint32_t d = (uint32_t)(k[j] >> shift) & 0xFF;
            pos[j] += L.lstart[d] + L.wcnt[w][d];
            L.stage[pos[j]] = k[j];
        }
    }
    // decoupled look-back over the per-digit counts of earlier tiles
    if (tid < RADIX) {
        const uint64_t ep = (uint64_t)epoch << 34;
        uint64_t *mine = status + (uint64_t)tile * RADIX + tid;
        uint32_t excl = 0;
        if (tile == 0) {
            st_status64(mine, ep | FLAG_INC | cnt);
        } else {
            st_status64(mine, ep | FLAG_AGG | cnt);
            // LOOKBACK tiles at a time: the tiles of a small call all start
            // together, and then a tile has about half the earlier ones to add
            int64_t j = (int64_t)tile - 1;
            uint32_t spins = 0;
            while (j >= 0) {
                uint64_t x[LOOKBACK];
#pragma unroll
                for (int b = 0; b < LOOKBACK; ++b)
                    x[b] = ld_status64(status + (uint64_t)(j >= b ? j - b : 0) * RADIX + tid);
                bool done = false, wait = false;
#pragma unroll
                for (int b = 0; b < LOOKBACK; ++b) {
                    if (done || wait || j < 0) continue;
                    if ((x[b] >> 34) != epoch || (x[b] & (FLAG_AGG | FLAG_INC)) == 0) {
                        wait = true;
                    } else {
                        excl += (uint32_t)x[b];
                        done = (x[b] & FLAG_INC) != 0;
                        --j;
                    }
                }
                if (done) break;
                if (wait) {
                    if (++spins > SPIN_LIMIT) {
                        atomicOr(err, DEV_ERR_LOOKBACK_TIMEOUT);
                        break;
                    }
                    __builtin_amdgcn_s_sleep(1);
                }
            }
            st_status64(mine, ep | FLAG_INC | (uint32_t)(excl + cnt));
        }
        L.gbase[tid] = start[tid] + excl - lst;
        // the last tile holds every digit's total: it must fill the digit's
        // range exactly (a caller's histogram that does not match the keys)
        if ((uint64_t)(tile + 1) * TILE >= n) {
            const uint32_t hi = tid + 1 < RADIX ? start[tid + 1] : (uint32_t)n;
            if (start[tid] + excl + cnt != hi) atomicOr(err, DEV_ERR_BAD_HIST);
        }
    }
    __syncthreads();
    const uint64_t left = n - base;
    const uint32_t n_tile = left < (uint64_t)TILE ? (uint32_t)left : (uint32_t)TILE;
    // keys out, remembering each slot's destination for the values (a
    // histogram that does not match the keys cannot send a write outside)
    uint32_t dst[ITEMS];
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const uint32_t i = (uint32_t)(tid + r * SORT_THREADS);
        dst[r] = NONE;
        if (i < n_tile) {
            const uint64_t kk = L.stage[i];
            dst[r] = L.gbase[(uint32_t)(kk >> shift) & 0xFF] + i;
            if (dst[r] < n) keys_out[dst[r]] = kk;
        }
    }
    __syncthreads();
    uint32_t *s_val = reinterpret_cast<uint32_t *>(L.stage);
#pragma unroll
    for (int j = 0; j < ITEMS; ++j)
        if (ok[j]) s_val[pos[j]] = v[j];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const uint32_t i = (uint32_t)(tid + r * SORT_THREADS);
        if (i < n_tile && dst[r] < n) vals_out[dst[r]] = s_val[i];
    }
    return true;
}

template <int ITEMS>
__global__ __launch_bounds__(SORT_THREADS, 4) void sort_pass_kernel(
    const uint64_t *__restrict__ keys_in, const uint32_t *__restrict__ vals_in,
    uint64_t *__restrict__ keys_out, uint32_t *__restrict__ vals_out, uint64_t n, int shift,
    const uint32_t *__restrict__ start, uint64_t *__restrict__ status, uint32_t *__restrict__ counter,
    uint32_t epoch, int32_t *__restrict__ err, const uint32_t *__restrict__ n_dev,
    const int32_t *__restrict__ gate) {
    if (gated_off(gate)) return;
    n = dev_count(n, n_dev);
    // Workgroups past the tile count take no tile (the counter then hands
    // out exactly the tiles there are) and leave at once: a grid sized for a
    // bound well above a device count costs little.
    if ((uint64_t)blockIdx.x * (ITEMS * SORT_THREADS) >= n) return;
    __shared__ SortLds<ITEMS> L;
    sort_tile(L, keys_in, vals_in, keys_out, vals_out, n, shift, start, status, counter, epoch, err);
}

// ---- links, and the way back to time order -------------------------------
// Equal neighbours in (key, t) order are consecutive uses of one key, giving
// the triple (t, prev(t), next(t)).  t is a permutation of [0, n), so the
// triples with t in [a, b) fill exactly positions [a, b) once they are
// partitioned by the top bits of t; the order inside a range does not matter
// because the last step places every triple at its own t.  Each partition
// pass therefore reserves its output runs with global atomics on per-bucket
// cursors (per workgroup chunk in the link, per tile later; see below)
// instead of a look-back, stages each tile digit-sorted in LDS and writes
// each run contiguously.
constexpr int LINK_THREADS = 256;
constexpr int LINK_ITEMS = 8;                          // link: 2048-element tiles
constexpr int LINK_TILE = LINK_THREADS * LINK_ITEMS;
constexpr int PART_THREADS = 512;
constexpr int PART_ITEMS = 16;                         // plain partition: 8192-element tiles
constexpr int PERM_TILE = PART_THREADS * PART_ITEMS;   // the larger tile
constexpr int PERM_RADIX = 1024;   // digits of a later pass (a tile spans two earlier buckets)
constexpr int LINK_RADIX = 256;    // digits of the first pass: at most 256 buckets
constexpr int PERM_LOCAL_BITS = 14;
constexpr uint64_t LINK_CHUNK_MAX = 1ull << 16;   // elements per workgroup, link

// Work per workgroup: a later pass takes one tile (it reserves per tile), the
// link, which reserves per chunk, chunks of up to 2^16 elements, eight per CU
// where n allows: four of its workgroups are on a CU at a time, so each place
// takes two chunks or more and ends with the others, and the runs that the
// workgroups in flight append to lie closer together (3.4e7 elements 337 us,
// with two chunks per CU 409).  The same on the host (grids) and the device (a
// count the GPU wrote).
constexpr int LINK_CHUNKS_PER_CU = 8;
__host__ __device__ inline uint64_t chunk_elems(uint64_t n, uint64_t chunks, uint64_t cap, uint64_t tile) {
    uint64_t c = (n + chunks - 1) / chunks;
    c = (c + tile - 1) / tile * tile;
    if (c > cap) c = cap;
    return c < tile ? tile : c;
}
__host__ __device__ inline uint64_t link_chunk(uint64_t n, int cus) {
    return chunk_elems(n, (uint64_t)cus * LINK_CHUNKS_PER_CU, LINK_CHUNK_MAX, LINK_TILE);
}
// Which tile of a later pass a workgroup takes: workgroups go to the eight XCDs
// in turn, and each XCD gets one contiguous eighth of the tiles.  Tiles that
// follow each other append to the same runs, and only within one XCD's L2 do
// their ends meet in the same line before it is written.  A grid of
// perm_grid(m) covers every count up to m; a tile past the last is none.
constexpr uint64_t XCDS = 8;
__host__ __device__ inline uint64_t perm_tiles(uint64_t n) { return (n + PERM_TILE - 1) / PERM_TILE; }
static unsigned perm_grid(uint64_t n) { return (unsigned)((perm_tiles(n) + XCDS - 1) / XCDS * XCDS); }
__device__ inline uint64_t perm_tile(uint64_t n, uint64_t block) {
    const uint64_t share = (perm_tiles(n) + XCDS - 1) / XCDS;
    return block / XCDS < share ? block % XCDS * share + block / XCDS : ~0ull;
}
// the most chunks any count up to n splits into (the grid of a pass)
static uint64_t max_chunks(uint64_t n, uint64_t chunk, uint64_t chunks, uint64_t cap) {
    const uint64_t by_cap = (n + cap - 1) / cap, at_n = (n + chunk - 1) / chunk;
    uint64_t g = by_cap > chunks + 1 ? by_cap : chunks + 1;
    if (at_n > g) g = at_n;
    return g;
}

// After the four passes over the low 32 key bits, equal keys are contiguous
// unless different keys share those bits ("mixed" runs, a few percent of the
// accesses for 64-bit hashes).  The link step resolves them by scanning the
// run: an element inside a block of equal keys finds its neighbour in one
// step, while a block boundary scans back (or forward) to the previous (next)
// block of its key or the run's end.  The scans of a workgroup share a budget
// of twice its element count; running out of it (adversarial keys: many keys
// sharing low bits) raises a flag that switches on the four passes over the
// high bits and a second link over the fully sorted keys, where equal keys
// are adjacent and no scan is needed.
__device__ __forceinline__ bool same_low(uint64_t a, uint64_t b) { return (uint32_t)a == (uint32_t)b; }

// Scan from position `from` (inclusive) in direction dir (-1 / +1) over
// elements sharing k's low bits; stop at k (found), at the run's end, or
// after `limit` steps.  Keys are read 8 at a time so a long scan costs one
// memory latency per 8 elements.  Returns false when the limit was reached
// first; *hit = position of k or UINT64_MAX.
constexpr int SCAN_BATCH = 8;
constexpr uint32_t LINK_SCAN_LIMIT = 64;   // memory steps a lane takes alone
__device__ __forceinline__ bool scan_run(const uint64_t *__restrict__ sk, uint64_t n, uint64_t k, uint64_t from,
                                         int dir, uint32_t limit, uint64_t *hit) {
    *hit = ~0ull;
    int64_t j = (int64_t)from;
    for (uint32_t steps = 0; steps < limit; steps += SCAN_BATCH) {
        uint64_t kb[SCAN_BATCH];
#pragma unroll
        for (int q = 0; q < SCAN_BATCH; ++q) {
            const int64_t x = j + dir * q;
            kb[q] = (x >= 0 && (uint64_t)x < n) ? sk[x] : ~k;   // ~k: differs from k in the low bits
        }
#pragma unroll
        for (int q = 0; q < SCAN_BATCH; ++q) {
            if (kb[q] == k) {
                *hit = (uint64_t)(j + dir * q);
                return true;
            }
            if (!same_low(kb[q], k)) return true;
        }
        j += dir * SCAN_BATCH;
    }
    return false;
}

// Previous (dir = -1) or next (dir = +1) element with the same full key as
// sorted position i, whose adjacent element shares the low key bits but not
// the key.  Lanes resolve such requests independently: each scans a few
// batches on its own; a lane still unresolved after that (a long run, e.g. a
// hot key sharing its low bits with another key) is taken over by the whole
// wave, 64 positions per step.  The wave steps are charged to the
// workgroup's budget (*budget, in positions); when it runs out the lane gives
// up and *overflow is raised, which switches on the passes over the high key
// bits and a second link.  All lanes of the wave must call this together.
__device__ __forceinline__ uint32_t resolve_mixed(const uint64_t *__restrict__ sk, const uint32_t *__restrict__ st,
                                                  uint64_t n, bool active, uint64_t i, int dir, int lane,
                                                  int32_t *budget, int32_t *__restrict__ overflow) {
    uint32_t res = NONE;
    uint64_t k = 0;
    int64_t cont = 0;
    bool need = false;
    if (active) {
        k = sk[i];
        const int64_t from = (int64_t)i + 2 * dir;   // i + dir is the known different key
        if (from >= 0 && (uint64_t)from < n) {
            uint64_t hit;
            if (scan_run(sk, n, k, (uint64_t)from, dir, LINK_SCAN_LIMIT, &hit)) {
                if (hit != ~0ull) res = st[hit];
            } else {
                need = true;
                cont = from + dir * (int64_t)LINK_SCAN_LIMIT;
            }
        }
    }
    for (uint64_t pending = ballot(need); pending; pending &= pending - 1) {
        const int L = __builtin_ctzll(pending);
        const uint64_t kL = shfl64(k, L);
        const int dL = __shfl(dir, L, WAVE);
        int64_t pos = (int64_t)shfl64((uint64_t)cont, L);
        uint32_t found = NONE;
        for (;;) {
            int32_t left = 0;
            if (lane == 0) left = atomicAdd(budget, -WAVE);
            left = __shfl(left, 0, WAVE);
            if (left < WAVE) {
                if (lane == 0) atomicOr(overflow, 1);
                break;
            }
            const int64_t x = pos + dL * lane;
            const uint64_t kk = (x >= 0 && (uint64_t)x < n) ? sk[x] : ~kL;
            const uint64_t hitm = ballot(kk == kL);
            const uint64_t ev = hitm | ballot(!same_low(kk, kL));
            if (ev) {
                const int f = __builtin_ctzll(ev);
                if ((hitm >> f) & 1) found = st[pos + dL * f];
                break;
            }
            pos += dL * WAVE;
        }
        if (lane == L) res = found;
    }
    return res;
}

// One workgroup owns a contiguous chunk of the input and streams it tile by
// tile: LDS counters give each element its slot inside its digit, the tile
// is staged digit-sorted in LDS (times, then (prev, next) pairs, through a
// single buffer), and each digit's part is appended to a run reserved in the
// bucket's output range.  The link reserves once per chunk: it first counts
// the chunk's digits and takes one run per digit with a single global atomic,
// so each bucket cursor sees one atomic per workgroup and the runs a
// workgroup appends to stay few and long.  Later passes skip that extra read
// of t and reserve per tile (their tiles are four times larger, so the runs
// stay long enough).  Longer tiles give longer runs per digit, hence fewer
// partially written lines; the link keeps 2048 because it holds keys and
// neighbours per element and waits on more loads: four small workgroups per
// CU overlap those waits better than two large.  A tile or chunk of a later
// pass spans at most 1024 consecutive buckets (see the plan), so digit =
// bucket mod 1024 names them without collision; the first pass has at most
// 256.
template <int TILE, int THREADS, int RADIX_N>
struct PermLds {
    uint64_t stage[TILE];   // bucket names while counting; per tile: times (as u32), then (prev, next) pairs
    uint32_t cnt[RADIX_N];
    uint32_t lstart[RADIX_N];
    uint32_t cur[RADIX_N];
    uint32_t tmp[THREADS / WAVE];
    int32_t budget;   // positions the link may still scan for long mixed runs
    uint32_t nmixed;  // mixed-run requests of the current tile (the list lives in `stage`)
};

template <bool FROM_SORT, int PERM_THREADS, int ITEMS, int RADIX_N, bool PER_TILE>
__device__ __forceinline__ void perm_partition_body(
    PermLds<PERM_THREADS * ITEMS, PERM_THREADS, RADIX_N> &L, const uint64_t *sk, const uint32_t *in_t,
    const uint64_t *in_pn, uint64_t n, int s, uint64_t chunk, uint64_t per_wg, uint32_t *cursor, uint32_t *out_t,
    uint64_t *out_pn, bool full, int32_t *overflow) {
    uint32_t *s_stage = reinterpret_cast<uint32_t *>(L.stage), *s_cnt = L.cnt, *s_lstart = L.lstart,
             *s_cur = L.cur, *s_bucket = reinterpret_cast<uint32_t *>(L.stage), *s_tmp = L.tmp;
    static_assert(RADIX_N % PERM_THREADS == 0 || PERM_THREADS % RADIX_N == 0, "whole digits per thread");
    // per-tile bucket names live in the stage buffer, which the link's
    // mixed-run list also uses
    static_assert(!(PER_TILE && FROM_SORT), "the link reserves per chunk");
    // digits per thread; with fewer digits than threads, threads below
    // RADIX_N own one digit each
    constexpr int DPT = RADIX_N >= PERM_THREADS ? RADIX_N / PERM_THREADS : 1;
    const bool owner = (int)threadIdx.x * DPT < RADIX_N;
    // positions fit 32 bits (n < 2^32 - 1); offsets from a tile's base are
    // compared against what is left, so nothing wraps near the end
    if (chunk * per_wg >= n) return;
    int tid0 = threadIdx.x;   // the tile loop below takes its own copy
    __asm__ volatile("" : "+v"(tid0));
    const uint32_t lo = (uint32_t)(chunk * per_wg);
    const uint32_t hi = (uint64_t)lo + per_wg < n ? (uint32_t)(lo + per_wg) : (uint32_t)n;

    // ---- (per chunk) count the chunk's digits and reserve one run per digit
    for (int i = tid0; i < RADIX_N; i += PERM_THREADS) s_cnt[i] = 0;
    if (tid0 == 0) L.budget = (int32_t)(2 * (hi - lo) + 4096);
    __syncthreads();
    if constexpr (!PER_TILE) {
    // eight loads in flight per thread before their LDS updates
    for (uint32_t b0 = lo; b0 < hi; b0 += 8 * PERM_THREADS) {
        const uint32_t left = hi - b0;
        uint32_t tt[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const uint32_t o = (uint32_t)(q * PERM_THREADS + tid0);
            tt[q] = o < left ? (in_t + b0)[o] : 0u;
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            // (a time outside [0, n) can only come from inconsistent input;
            // it reserves nothing and its element is not written)
            if ((uint32_t)(q * PERM_THREADS + tid0) < left && tt[q] < n) {
                const uint32_t d = (tt[q] >> s) & (RADIX_N - 1);
                atomicAdd(&s_cnt[d], 1u);
                s_bucket[d] = tt[q] >> s;   // every writer of digit d writes the same bucket
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < DPT && owner; ++q) {
        const int d = tid0 * DPT + q;
        const uint32_t c = s_cnt[d];
        if (c) s_cur[d] = (s_bucket[d] << s) + atomicAdd(&cursor[s_bucket[d]], c);
    }
    __syncthreads();
    }

    // ---- stream the chunk tile by tile
    constexpr int TILE = PERM_THREADS * ITEMS;
    for (uint32_t base = lo; base < hi; base += TILE) {
        const uint32_t left = hi - base;
        // an opaque copy of the thread index: values derived from it are
        // recomputed per tile instead of being held (and spilled) across the loop
        int tid = threadIdx.x;
        __asm__ volatile("" : "+v"(tid));
        const int lane = tid & (WAVE - 1);
        for (int i = tid; i < RADIX_N; i += PERM_THREADS) s_cnt[i] = 0;
        if (tid == 0) L.nmixed = 0;
        __syncthreads();
        // per-tile base pointers keep the per-lane offsets 32-bit.  Every
        // load of the tile is issued before the first use, so a tile costs
        // one memory latency, not one per item.
        const uint32_t *tb = in_t + base;
        uint32_t t[ITEMS], pos[ITEMS];
        uint64_t pn[ITEMS];   // prev | next << 32
        bool ok[ITEMS];
        if (FROM_SORT) {
            const uint64_t *kb = sk + base;
            const int w = tid / WAVE;
            uint64_t k[ITEMS];
#pragma unroll
            for (int j = 0; j < ITEMS; ++j) {
                const uint32_t o = (uint32_t)(j * PERM_THREADS + tid);
                ok[j] = o < left;
                const uint32_t oc = ok[j] ? o : 0u;
                t[j] = tb[oc];
                k[j] = kb[oc];
            }
            // the elements just outside each item's wave: lane j loads the
            // one before item j's first lane, lane 8 + j the one after its
            // last valid lane
            uint64_t ek = 0;
            uint32_t et = 0;
            {
                const int j = lane & 7;
                const uint32_t w0 = (uint32_t)(j * PERM_THREADS + w * WAVE);   // wave's first offset
                const uint32_t lastj = w0 < left ? (left - 1 - w0 < (uint32_t)(WAVE - 1) ? left - 1 - w0 : WAVE - 1) : 0u;
                const uint64_t gp = lane < 8 ? (uint64_t)base + w0 - 1 : (uint64_t)base + w0 + lastj + 1;
                const bool want = lane < 16 && w0 < left && (lane < 8 ? (uint64_t)base + w0 > 0 : gp < n);
                if (want) {
                    ek = sk[gp];
                    et = in_t[gp];
                }
            }
            // fast links from neighbours; a lane whose neighbour shares the
            // low bits but not the key appends a request (offset, direction)
            // to the tile's list, resolved below by the whole workgroup
            uint32_t *mlist = reinterpret_cast<uint32_t *>(L.stage);   // 2 * TILE entries
            uint32_t mixbits = 0;   // bit 2j: item j's prev is in the list, bit 2j+1: its next
#pragma unroll
            for (int j = 0; j < ITEMS; ++j) {
                const uint32_t o = (uint32_t)(j * PERM_THREADS + tid);
                const uint64_t i = (uint64_t)base + o;
                // consecutive lanes hold consecutive sorted positions: the
                // neighbours' keys and times come from the adjacent lanes
                const uint32_t w0 = o - (uint32_t)lane;
                const int last = w0 < left ? (int)(left - 1 - w0 < (uint32_t)(WAVE - 1) ? left - 1 - w0 : WAVE - 1)
                                           : -1;
                uint64_t kp = from_lower64(k[j]), kn = from_upper64(k[j]);
                uint32_t tp = from_lower(t[j]);
                uint32_t tn = from_upper(t[j]);
                const uint64_t ekp = readlane64(ek, j), ekn = readlane64(ek, 8 + j);
                const uint32_t etp = (uint32_t)__builtin_amdgcn_readlane((int)et, j);
                const uint32_t etn = (uint32_t)__builtin_amdgcn_readlane((int)et, 8 + j);
                bool mp = false, mn = false;
                uint32_t pv = NONE, nx = NONE;
                if (ok[j]) {
                    const bool has_next = i + 1 < n;
                    if (lane == 0) { kp = ekp; tp = etp; }
                    if (lane == last) { kn = ekn; tn = etn; }
                    if (i > 0 && kp == k[j]) pv = tp;
                    else mp = i > 0 && !full && same_low(kp, k[j]);
                    if (has_next && kn == k[j]) nx = tn;
                    else mn = has_next && !full && same_low(kn, k[j]);
                }
                const uint64_t mpm = ballot(mp), mnm = ballot(mn);
                if (mpm | mnm) {
                    const uint32_t cnt = (uint32_t)__popcll(mpm) + (uint32_t)__popcll(mnm);
                    uint32_t e0 = 0;
                    if (lane == 0) e0 = atomicAdd(&L.nmixed, cnt);
                    e0 = (uint32_t)__shfl((int)e0, 0, WAVE);
                    if (mp) {
                        const uint32_t e = e0 + mbcnt(mpm);
                        mlist[e] = o << 1;
                        pv = e;
                        mixbits |= 1u << (2 * j);
                    }
                    if (mn) {
                        const uint32_t e = e0 + (uint32_t)__popcll(mpm) + mbcnt(mnm);
                        mlist[e] = (o << 1) | 1u;
                        nx = e;
                        mixbits |= 2u << (2 * j);
                    }
                }
                pn[j] = (uint64_t)pv | ((uint64_t)nx << 32);
            }
            __syncthreads();
            const uint32_t nm = L.nmixed;
            if (nm) {
                // resolve the list in place (entry -> time of the neighbour)
                for (uint32_t e0 = 0; e0 < nm; e0 += PERM_THREADS) {
                    const uint32_t e = e0 + tid;
                    const bool act = e < nm;
                    const uint32_t code = act ? mlist[e] : 0u;
                    const uint32_t res = resolve_mixed(sk, in_t, n, act, (uint64_t)base + (code >> 1),
                                                       (code & 1) ? 1 : -1, lane, &L.budget, overflow);
                    if (act) mlist[e] = res;
                }
                __syncthreads();
#pragma unroll
                for (int j = 0; j < ITEMS; ++j) {
                    if (mixbits & (3u << (2 * j))) {
                        uint32_t pv = (uint32_t)pn[j], nx = (uint32_t)(pn[j] >> 32);
                        if (mixbits & (1u << (2 * j))) pv = mlist[pv];
                        if (mixbits & (2u << (2 * j))) nx = mlist[nx];
                        pn[j] = (uint64_t)pv | ((uint64_t)nx << 32);
                    }
                }
            }
        } else {
#pragma unroll
            for (int j = 0; j < ITEMS; ++j) {
                const uint32_t o = (uint32_t)(j * PERM_THREADS + tid);
                ok[j] = o < left;
                const uint32_t oc = ok[j] ? o : 0u;
                t[j] = tb[oc];
                pn[j] = (in_pn + base)[oc];
            }
        }
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) {
            // (per tile: a time outside [0, n), from inconsistent input,
            // reserves nothing and is not written)
            if (PER_TILE) ok[j] = ok[j] && t[j] < n;
            if (ok[j]) {
                pos[j] = atomicAdd(&s_cnt[(t[j] >> s) & (RADIX_N - 1)], 1u);
                if (PER_TILE) s_bucket[(t[j] >> s) & (RADIX_N - 1)] = t[j] >> s;
            }
        }
        __syncthreads();
        uint32_t c[DPT], mine = 0, total;
#pragma unroll
        for (int q = 0; q < DPT; ++q) {
            c[q] = owner ? s_cnt[tid * DPT + q] : 0u;
            mine += c[q];
        }
        uint32_t run = block_excl_scan(mine, s_tmp, &total);
#pragma unroll
        for (int q = 0; q < DPT && owner; ++q) {
            s_lstart[tid * DPT + q] = run;
            run += c[q];
            if (PER_TILE && c[q]) {
                const uint32_t b = s_bucket[tid * DPT + q];
                s_cur[tid * DPT + q] = (b << s) + atomicAdd(&cursor[b], c[q]);
            }
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) {
            if (!ok[j]) continue;
            pos[j] += s_lstart[(t[j] >> s) & (RADIX_N - 1)];
            s_stage[pos[j]] = t[j];
        }
        __syncthreads();
        // times out, remembering each slot's destination for the (prev, next) pairs
        uint32_t dst[ITEMS];
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) {
            const uint32_t slot = (uint32_t)(tid + r * PERM_THREADS);
            dst[r] = ~0u;
            if (slot < total) {
                const uint32_t tt = s_stage[slot];
                const uint32_t d = (tt >> s) & (RADIX_N - 1);
                dst[r] = s_cur[d] + (slot - s_lstart[d]);
                if (dst[r] < n) out_t[dst[r]] = tt;
            }
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < ITEMS; ++j)
            if (ok[j]) L.stage[pos[j]] = pn[j];
        __syncthreads();
#pragma unroll
        for (int r = 0; r < ITEMS; ++r)
            if (dst[r] < n) out_pn[dst[r]] = L.stage[tid + r * PERM_THREADS];
        if (!PER_TILE)
#pragma unroll
            for (int q = 0; q < DPT; ++q)
                if (owner) s_cur[tid * DPT + q] += c[q];
        __syncthreads();
    }
}

// The link variant holds more state per element (keys and neighbours): four
// 256-thread workgroups per CU; the plain partition runs two of 512.  The link
// over keys sorted by their low 32 bits raises *flag when a mixed run is too
// long to scan.
__global__ __launch_bounds__(LINK_THREADS, 4) void link_partition_kernel(
    const uint64_t *__restrict__ sk, const uint32_t *__restrict__ in_t, uint64_t n, int s, int cus,
    uint32_t *__restrict__ cursor, uint32_t *__restrict__ out_t, uint64_t *__restrict__ out_pn,
    int32_t *__restrict__ flag, const uint32_t *__restrict__ n_dev, const int32_t *__restrict__ gate) {
    if (gated_off(gate)) return;
    n = dev_count(n, n_dev);
    const uint64_t per_wg = link_chunk(n, cus);
    __shared__ PermLds<LINK_TILE, LINK_THREADS, LINK_RADIX> L;
    perm_partition_body<true, LINK_THREADS, LINK_ITEMS, LINK_RADIX, false>(L, sk, in_t, nullptr, n, s, blockIdx.x,
                                                                           per_wg, cursor, out_t, out_pn, false, flag);
}

// Bound: the writes, whose runs are a few lines long.  One tile per workgroup,
// an XCD's tiles contiguous: two launches over 9.4e7 elements in all 511 us
// (4.4 TB/s of 24 bytes each), in the order of the workgroups 580, as two
// chunks per CU 648.
__global__ __launch_bounds__(PART_THREADS, 4) void perm_partition_kernel(
    const uint32_t *__restrict__ in_t, const uint64_t *__restrict__ in_pn, uint64_t n, int s,
    uint32_t *__restrict__ cursor, uint32_t *__restrict__ out_t, uint64_t *__restrict__ out_pn,
    const uint32_t *__restrict__ n_dev, const int32_t *__restrict__ gate) {
    if (gated_off(gate)) return;
    n = dev_count(n, n_dev);
    const uint64_t tile = perm_tile(n, blockIdx.x);
    if (tile >= perm_tiles(n)) return;
    __shared__ PermLds<PERM_TILE, PART_THREADS, PERM_RADIX> L;
    perm_partition_body<false, PART_THREADS, PART_ITEMS, PERM_RADIX, true>(L, nullptr, in_t, in_pn, n, s, tile,
                                                                           PERM_TILE, cursor, out_t, out_pn, true,
                                                                           nullptr);
}

// every 16384-range of t holds exactly its own triples: place the (prev,
// next) pairs by t in LDS (128 KB, one 1024-thread workgroup per CU) and
// write prev / next in time order
constexpr int LOCAL_THREADS = 1024;
__global__ __launch_bounds__(LOCAL_THREADS) void perm_local_kernel(const uint32_t *__restrict__ in_t,
                                                                   const uint64_t *__restrict__ in_pn,
                                                                   uint64_t n, uint32_t *__restrict__ prev,
                                                                   uint32_t *__restrict__ next,
                                                                   const int32_t *__restrict__ hdr, SortReport report,
                                                                   const uint32_t *__restrict__ n_dev,
                                                                   const int32_t *__restrict__ gate) {
    constexpr uint32_t SPAN = 1u << PERM_LOCAL_BITS;
    constexpr int PER = SPAN / LOCAL_THREADS;
    __shared__ uint64_t s_pn[SPAN];
    if (gated_off(gate)) return;
    if (report.hdr && blockIdx.x == 0 && threadIdx.x == 0) {
        if (hdr[0]) atomicOr(report.hdr, hdr[0]);
        report.hdr[report.high_word] = hdr[1];
    }
    n = dev_count(n, n_dev);
    // one range per workgroup, or several from a capped grid
    for (uint64_t r0 = (uint64_t)blockIdx.x * SPAN; r0 < n; r0 += (uint64_t)gridDim.x * SPAN) {
        const uint32_t cnt = n - r0 < SPAN ? (uint32_t)(n - r0) : SPAN;
        const uint32_t *tb = in_t + r0;
        const uint64_t *pb = in_pn + r0;
        uint32_t tt[PER];
        uint64_t v[PER];
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const uint32_t j = threadIdx.x + q * LOCAL_THREADS;
            const uint32_t jc = j < cnt ? j : 0u;
            tt[q] = tb[jc];
            v[q] = pb[jc];
        }
#pragma unroll
        for (int q = 0; q < PER; ++q)
            if (threadIdx.x + q * LOCAL_THREADS < cnt) s_pn[(uint32_t)(tt[q] - r0) & (SPAN - 1)] = v[q];
        __syncthreads();
        for (uint32_t j = threadIdx.x; j < cnt; j += LOCAL_THREADS) {
            const uint64_t x = s_pn[j];
            prev[r0 + j] = (uint32_t)x;
            next[r0 + j] = (uint32_t)(x >> 32);
        }
        __syncthreads();   // the range has left the LDS before the next one comes in
    }
}

// Partition plan for the way back to time order.  The last step uses
// 16384-ranges of t.  The link splits into at most 256 buckets, later passes
// into at most 512 per earlier bucket.  Every bucket is at least 16384 wide,
// so a tile of a later pass (8192 elements) spans at most two earlier
// buckets, i.e. at most 1024 consecutive buckets of its own pass, and
// (bucket mod 1024) names them without collision inside the tile.
struct PermPlan {
    int passes;
    int s[4];
    uint64_t buckets[4];
    uint64_t max_buckets;
};

static PermPlan plan_perm(uint64_t n) {
    PermPlan p{};
    int nbits = 0;
    while (nbits < 64 && (1ull << nbits) < n) ++nbits;
    int cur = nbits;
    int shifts[4], k = 0;
    // Up to 8 bits in the link (its tiles are small), up to 9 in later passes:
    // longer runs per tile and bucket than 10.  With one later pass the link
    // takes half of the bits, for the same reason (3.4e7 elements, 12 bits: link
    // and later pass 278 + 214 us, as 8 and 4 bits 337 + 206, both with the
    // later pass as two chunks per CU; it takes 188 now).
    const int total = nbits - PERM_LOCAL_BITS;
    int width = 8;
    if (total > 8 && total < 15) width = (total + 1) / 2;
    while (cur > PERM_LOCAL_BITS && k < 4) {
        int next_s = cur - width > PERM_LOCAL_BITS ? cur - width : PERM_LOCAL_BITS;
        shifts[k++] = next_s;
        cur = next_s;
        width = 9;
    }
    if (k == 0) shifts[k++] = PERM_LOCAL_BITS;
    p.passes = k;
    p.max_buckets = 1;
    for (int i = 0; i < k; ++i) {
        p.s[i] = shifts[i];
        p.buckets[i] = (n + (1ull << shifts[i]) - 1) >> shifts[i];
        if (p.buckets[i] > p.max_buckets) p.max_buckets = p.buckets[i];
    }
    return p;
}

// The control block: histograms, counters and partition cursors (one array per
// partition: both links, then the later passes), contiguous so that one fill
// clears them, and the digit starts.
static SortCtl take_ctl(Carver &c, uint64_t n) {
    SortCtl k;
    const PermPlan pp = plan_perm(n);
    k.hdr = c.take<int32_t>(WS_HEADER / sizeof(int32_t));
    k.start = c.take<uint32_t>(SORT_PASSES * RADIX);
    const size_t z0 = c.off;
    k.hist = c.take<uint32_t>(SORT_PASSES * RADIX);
    k.words = c.take<uint32_t>(CTL_WORDS);
    k.link2 = c.take<uint32_t>(LINK_RADIX);
    for (int i = 0; i < pp.passes; ++i) k.cursor[i] = c.take<uint32_t>(pp.buckets[i]);
    k.zero_words = (c.off - z0) / sizeof(uint32_t);
    return k;
}
SortCtl sort_ctl(void *at, uint64_t n, size_t *bytes) {
    Carver c{(char *)at, 0};
    const SortCtl k = take_ctl(c, n);
    *bytes = c.off;
    return k;
}
void sort_ctl_clear(Fills &f, const SortCtl &k) {
    f.add(k.hdr, 0u, 2);
    f.add(k.hist, 0u, k.zero_words);
}

// tiles of a sort pass over n keys
static uint64_t pass_tiles(uint64_t n) {
    const uint64_t t = n <= SORT_MAX_4 ? 4 * SORT_THREADS : n <= SORT_MAX_8 ? 8 * SORT_THREADS : SORT_TILE;
    return (n + t - 1) / t;
}
struct SortBufs {
    uint64_t *k1, *k2;   // sort ping-pong; afterwards (prev, next) pairs
    uint32_t *v1, *v2;   // sort ping-pong; afterwards times t
    uint64_t *status;
};
static SortBufs take_bufs(Carver &c, uint64_t n) {
    SortBufs b;
    b.k1 = c.take<uint64_t>(n);
    b.k2 = c.take<uint64_t>(n);
    b.v1 = c.take<uint32_t>(n);
    b.v2 = c.take<uint32_t>(n);
    // (at least the smaller tiles' words, so that a larger n never needs less)
    uint64_t tiles = pass_tiles(n);
    for (const uint64_t m : {SORT_MAX_4, SORT_MAX_8})
        if (n > m && tiles < pass_tiles(m)) tiles = pass_tiles(m);
    b.status = c.take<uint64_t>(tiles * RADIX);
    return b;
}
size_t sort_bufs_bytes(uint64_t n) {
    Carver c{nullptr, 0};
    take_bufs(c, n);
    return c.off;
}

// ---- the whole of prev/next, or its tail, in one launch ------------------
// A path that a call seldom takes (the passes over the high key bits; the
// generic path behind the chained one) must still be enqueued, since the
// choice is made on the device, and a launch that its gate turns off costs
// about 4.5 us in the stream: eight launches for the high bits and twenty for
// the generic path.  Here they are one persistent kernel of phases (for the
// generic path, where that is the better one: prev_next_rare).  A phase
// hands out its chunks from a counter and counts the finished ones; a
// workgroup goes on to the next phase once all are finished.  Only running
// workgroups hold chunks, so the wait ends whatever part of the grid is
// resident.
enum SortPhase {
    PH_HIST,
    PH_PASS,
    PH_LINK = PH_PASS + 4,
    PH_HIST2,
    PH_PASS2,
    PH_LINK2 = PH_PASS2 + 4,
    PH_PERM,
    PH_COUNT = PH_PERM + 3
};
static_assert(CTL_PHASE + 2 * PH_COUNT <= CTL_WORDS, "the control words hold every phase");

struct SortJob {
    const uint64_t *keys;
    uint64_t n;
    const uint32_t *n_dev;
    const uint32_t *key_hist;
    SortCtl k;
    SortBufs b;
    PermPlan plan;
    int cus;
    bool whole;   // from the first pass to the last partition; else only the high bits and the second link
    RareGate rare;
};

union PersistentLds {
    SortLds<SORT_ITEMS> sort;
    PermLds<LINK_TILE, SORT_THREADS, LINK_RADIX> link;
    PermLds<PERM_TILE, PART_THREADS, PERM_RADIX> perm;
    uint32_t hist[HIST_DIGITS * RADIX];
};
static_assert(SORT_THREADS == PART_THREADS, "one workgroup size for all phases");

// the next chunk of a phase, for the whole workgroup
__device__ __forceinline__ uint32_t next_chunk(uint32_t *ctl, int phase, uint32_t *s_word) {
    __syncthreads();
    if (threadIdx.x == 0) *s_word = atomicAdd(&ctl[CTL_PHASE + 2 * phase], 1u);
    __syncthreads();
    return *s_word;
}
__device__ __forceinline__ uint32_t *phase_done(uint32_t *ctl, int phase) { return &ctl[CTL_PHASE + 2 * phase + 1]; }

// histograms of four byte digits from p0 on, then their starts; `clear`: the
// look-back status is cleared on the way, `given`: the histograms are known
__device__ __forceinline__ void persistent_hist(const SortJob &j, uint64_t n, int p0, int phase, bool clear,
                                                const uint32_t *given, PersistentLds &L, uint32_t *s_tmp,
                                                uint32_t *s_word) {
    // a chunk is whole tiles: two per workgroup, up to eight (a chunk ends with
    // a flush of its histogram to device memory)
    const uint64_t tiles = (n + SORT_TILE - 1) / SORT_TILE, even = tiles / (2 * gridDim.x);
    const uint64_t per = even < 1 ? 1 : even > 8 ? 8 : even, CHUNK = per * SORT_TILE, WORDS = per * RADIX;
    const uint64_t words = tiles * RADIX;
    const uint32_t chunks = (uint32_t)((tiles + per - 1) / per);
    uint32_t mine = 0;
    for (uint32_t c; (c = next_chunk(j.k.words, phase, s_word)) < chunks; ++mine) {
        const uint64_t lo = (uint64_t)c * CHUNK, hi = lo + CHUNK < n ? lo + CHUNK : n;
        if (clear)
            for (uint64_t i = c * WORDS + threadIdx.x; i < (c + 1) * WORDS && i < words; i += SORT_THREADS)
                j.b.status[i] = 0;
        if (!given) digit_hist(j.keys, lo, hi, blockDim.x, p0, L.hist, j.k.hist);
    }
    finish_phase(phase_done(j.k.words, phase), mine, chunks, j.k.hdr);
    // every workgroup works the starts out and writes the same words
    digit_starts(given ? given : j.k.hist + p0 * RADIX, j.k.start + p0 * RADIX, n, s_tmp, j.k.hdr);
    __threadfence_block();
    __syncthreads();
}

// the verdict of the path that a rare one stands behind
__device__ __forceinline__ int32_t rare_reason(const RareGate &r) {
    if (*r.good == 0) return *r.reason;
    return *r.error ? r.error_reason : *r.fail ? r.fail_reason : 0;
}
__global__ void rare_gate_kernel(RareGate r) {
    const int32_t why = rare_reason(r);
    if (why == 0) return;
    *r.reason = why;
    *r.on = 1;
}

__global__ __launch_bounds__(SORT_THREADS, 4) void sort_persistent_kernel(SortJob j, const int32_t *gate) {
    if (gated_off(gate)) return;
    if (j.whole) {
        const int32_t why = rare_reason(j.rare);
        if (why == 0) return;
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            *j.rare.reason = why;
            *j.rare.on = 1;
        }
    } else if (j.k.hdr[1] == 0) {
        return;
    }
    const uint64_t n = dev_count(j.n, j.n_dev);
    __shared__ PersistentLds L;
    __shared__ uint32_t s_tmp[SORT_THREADS / WAVE], s_word;
    uint32_t *ctl = j.k.words;
    const uint32_t tiles = (uint32_t)((n + SORT_TILE - 1) / SORT_TILE);
    auto pass = [&](int p) {
        const uint64_t *kin = p == 0 ? j.keys : (p & 1) ? j.b.k1 : j.b.k2;
        const uint32_t *vin = p == 0 ? nullptr : (p & 1) ? j.b.v1 : j.b.v2;
        uint64_t *kout = (p & 1) ? j.b.k2 : j.b.k1;
        uint32_t *vout = (p & 1) ? j.b.v2 : j.b.v1;
        const int phase = p < SORT_PASSES / 2 ? PH_PASS + p : PH_PASS2 + p - SORT_PASSES / 2;
        uint32_t mine = 0;
        __syncthreads();
        while (sort_tile(L.sort, kin, vin, kout, vout, n, 8 * p, j.k.start + p * RADIX, j.b.status,
                         ctl + CTL_TILE + p, (uint32_t)(p + 1), j.k.hdr)) {
            ++mine;
            __syncthreads();   // the tile has left the LDS before the next one comes in
        }
        finish_phase(phase_done(ctl, phase), mine, tiles, j.k.hdr);
    };
    auto link = [&](int phase, uint32_t *cursor, bool full) {
        const uint64_t per = link_chunk(n, j.cus);
        const uint32_t chunks = (uint32_t)((n + per - 1) / per);
        uint32_t mine = 0;
        for (uint32_t c; (c = next_chunk(ctl, phase, &s_word)) < chunks; ++mine)
            perm_partition_body<true, SORT_THREADS, LINK_TILE / SORT_THREADS, LINK_RADIX, false>(
                L.link, j.b.k2, j.b.v2, nullptr, n, j.plan.s[0], c, per, cursor, j.b.v1, j.b.k1, full,
                full ? nullptr : j.k.hdr + 1);
        finish_phase(phase_done(ctl, phase), mine, chunks, j.k.hdr);
    };
    if (j.whole) {
        persistent_hist(j, n, 0, PH_HIST, true, j.key_hist, L, s_tmp, &s_word);
#pragma unroll 1
        for (int p = 0; p < SORT_PASSES / 2; ++p) pass(p);
        link(PH_LINK, j.k.cursor[0], false);
    }
    // (the flag is only ever raised, before the phase that precedes this ends)
    if (__hip_atomic_load(j.k.hdr + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
        persistent_hist(j, n, SORT_PASSES / 2, PH_HIST2, false, nullptr, L, s_tmp, &s_word);
        // the passes go on from the low-sorted keys (k2, v2); the first link's
        // triples in (k1, v1) are overwritten and made again
#pragma unroll 1
        for (int p = SORT_PASSES / 2; p < SORT_PASSES; ++p) pass(p);
        link(PH_LINK2, j.k.link2, true);
    }
    if (j.whole) {
#pragma unroll 1
        for (int i = 1; i < j.plan.passes; ++i) {
            const uint32_t chunks = (uint32_t)perm_tiles(n);
            // (selected, not indexed: the job stays out of scratch memory)
            const bool odd = i & 1;
            const int shift = i == 1 ? j.plan.s[1] : i == 2 ? j.plan.s[2] : j.plan.s[3];
            uint32_t *cursor = i == 1 ? j.k.cursor[1] : i == 2 ? j.k.cursor[2] : j.k.cursor[3];
            uint32_t mine = 0;
            for (uint32_t c; (c = next_chunk(ctl, PH_PERM + i - 1, &s_word)) < chunks; ++mine)
                perm_partition_body<false, PART_THREADS, PART_ITEMS, PERM_RADIX, true>(
                    L.perm, nullptr, odd ? j.b.v1 : j.b.v2, odd ? j.b.k1 : j.b.k2, n, shift, c, PERM_TILE, cursor,
                    odd ? j.b.v2 : j.b.v1, odd ? j.b.k2 : j.b.k1, true, nullptr);
            finish_phase(phase_done(ctl, PH_PERM + i - 1), mine, chunks, j.k.hdr);
        }
    }
}

// Workgroups of the persistent launch: one per sort tile, and in small calls one
// per link tile, which are shorter, up to 32: the link's scans of keys that
// share their low bits would wait for a few workgroups (a chained call over
// 2.0e4 such keys 0.70 ms, with three workgroups 1.46; over 1.0e6 random keys
// one per link tile, 489, takes 0.46 and one per sort tile 0.27).
constexpr uint64_t PERSISTENT_MIN = 32;
static unsigned persistent_grid(uint64_t n) {
    const uint64_t tiles = (n + SORT_TILE - 1) / SORT_TILE, links = (n + LINK_TILE - 1) / LINK_TILE;
    const uint64_t few = links < PERSISTENT_MIN ? links : PERSISTENT_MIN;
    return capped(tiles < few ? few : tiles, 2);
}

static pc_status perm_local(const SortJob &j, uint32_t *prev, uint32_t *next, hipStream_t s, const int32_t *gate,
                            const SortReport &report) {
    const int cur = (j.plan.passes - 1) & 1;
    const uint64_t span = 1ull << PERM_LOCAL_BITS;
    const uint64_t ranges = (j.n + span - 1) / span;
    PC_LAUNCH(K_PERM_LOCAL, perm_local_kernel, dim3(j.whole ? capped(ranges, 1) : (unsigned)ranges),
              dim3(LOCAL_THREADS), 0, s, cur ? j.b.v2 : j.b.v1, cur ? j.b.k2 : j.b.k1, j.n, prev, next,
              (const int32_t *)j.k.hdr, report, j.n_dev, gate);
    return PC_OK;
}

pc_status prev_next_core(const uint64_t *keys, uint64_t n, const uint32_t *n_dev, uint32_t *prev, uint32_t *next,
                         const uint32_t *key_hist, const SortCtl &k, void *bufs, hipStream_t s, const int32_t *gate,
                         const SortReport &report) {
    Carver c{(char *)bufs, 0};
    const SortBufs b = take_bufs(c, n);
    if (n == 0) return PC_OK;
    const uint64_t tiles = pass_tiles(n);
    const int cus = device_cus();
    // The plan is made for the bound n: with fewer elements its later buckets
    // stay empty.
    const PermPlan pp = plan_perm(n);
    if (pp.buckets[0] > (uint64_t)LINK_RADIX) return PC_ERR_TOO_LARGE;   // the plan never splits wider
    Fills f;
    sort_ctl_clear(f, k);
    f.add(b.status, 0u, tiles * RADIX * 2);
    PC_LAUNCH(K_FILL32, sort_init_kernel, dim3(fill_blocks(f)), dim3(256), 0, s, f, key_hist, k.start, n, k.hdr, n_dev,
              gate);
    uint64_t hg = (n + 4095) / 4096;
    if (hg > (uint64_t)cus) hg = (uint64_t)cus;
    // the low bytes' histograms: handed in by the hash, or counted here
    if (!key_hist)
        PC_LAUNCH(K_SORT_HIST, sort_hist_kernel, dim3((unsigned)hg), dim3(HIST_THREADS), 0, s, keys, n, k.hist, k.start,
                  k.words, k.hdr, n_dev, gate);
    const uint64_t *kin = keys;
    const uint32_t *vin = nullptr;
    for (int p = 0; p < SORT_PASSES / 2; ++p) {
        uint64_t *kout = (p & 1) ? b.k2 : b.k1;
        uint32_t *vout = (p & 1) ? b.v2 : b.v1;
        const auto pass = n <= SORT_MAX_4   ? sort_pass_kernel<4>
                          : n <= SORT_MAX_8 ? sort_pass_kernel<8>
                                            : sort_pass_kernel<SORT_ITEMS>;
        PC_LAUNCH(K_SORT_PASS, pass, dim3((unsigned)tiles), dim3(SORT_THREADS), 0, s, kin, vin, kout, vout, n, 8 * p,
                  k.start + p * RADIX, b.status, k.words + CTL_TILE + p, (uint32_t)(p + 1), k.hdr, n_dev, gate);
        kin = kout;
        vin = vout;
    }
    // Links + partition back to time order.  The sort leaves (key, t) in
    // (k2, v2) after four passes and again after eight; the triples ping-pong
    // between the first sort buffers ((prev, next) pairs in k1, t in v1) and,
    // once the sorted keys have been consumed, the second ones (k2, v2).
    const unsigned ltiles =
        (unsigned)max_chunks(n, link_chunk(n, cus), (uint64_t)cus * LINK_CHUNKS_PER_CU, LINK_CHUNK_MAX);
    PC_LAUNCH(K_LINK, link_partition_kernel, dim3(ltiles), dim3(LINK_THREADS), 0, s, kin, vin, n, pp.s[0], cus,
              k.cursor[0], b.v1, b.k1, k.hdr + 1, n_dev, gate);
    // the passes over the high bits and a second link, if the first one met a
    // mixed run too long to scan (header word 1)
    const SortJob j{keys, n, n_dev, key_hist, k, b, pp, cus, false, RareGate{}};
    PC_LAUNCH(K_SORT_HIGH, sort_persistent_kernel, dim3(persistent_grid(n)), dim3(SORT_THREADS), 0, s,
              j, gate);
    uint32_t *bt[2] = {b.v1, b.v2};
    uint64_t *bpn[2] = {b.k1, b.k2};
    for (int i = 1; i < pp.passes; ++i) {
        const int from = (i - 1) & 1;
        PC_LAUNCH(K_PERM, perm_partition_kernel, dim3(perm_grid(n)), dim3(PART_THREADS), 0, s, bt[from], bpn[from], n,
                  pp.s[i], k.cursor[i], bt[from ^ 1], bpn[from ^ 1], n_dev, gate);
    }
    return perm_local(j, prev, next, s, gate, report);
}

// As one persistent launch, or as the launches of prev_next_core behind the
// verdict.  On, a chained call over random keys took 0.23 ms persistent at
// 1.0e5 keys, 0.33 as launches; 0.63 and 0.37 at 3.0e6; 2.61 and 2.02 at
// 3.0e7; 13.3 and 12.2 at 2.0e8: the ends of the phases weigh most where a
// phase is a few tiles per CU.  Off, which is the rule, the launches cost 27 us
// more than the one at 2.8e7 keys (of a step of 1.76 ms), and with their
// grids' size 0.37 ms of 20.4 at 8.0e8, so the largest calls keep the one.
constexpr uint64_t RARE_LAUNCHES_MIN = 1ull << 20, RARE_LAUNCHES_MAX = 1ull << 26;
pc_status prev_next_rare(const uint64_t *keys, uint64_t n, uint32_t *prev, uint32_t *next, const uint32_t *key_hist,
                         const SortCtl &k, void *bufs, hipStream_t s, const RareGate &rare, const SortReport &report) {
    if (n >= RARE_LAUNCHES_MIN && n < RARE_LAUNCHES_MAX) {
        PC_LAUNCH(K_FILL32, rare_gate_kernel, dim3(1), dim3(1), 0, s, rare);
        return prev_next_core(keys, n, nullptr, prev, next, key_hist, k, bufs, s, rare.on, report);
    }
    Carver c{(char *)bufs, 0};
    const PermPlan pp = plan_perm(n);
    if (pp.buckets[0] > (uint64_t)LINK_RADIX) return PC_ERR_TOO_LARGE;
    const SortJob j{keys, n, nullptr, key_hist, k, take_bufs(c, n), pp, device_cus(), true, rare};
    PC_LAUNCH(K_SORT_HIGH, sort_persistent_kernel, dim3(persistent_grid(n)), dim3(SORT_THREADS), 0, s, j,
              (const int32_t *)nullptr);
    return perm_local(j, prev, next, s, rare.on, report);
}

}  // namespace pc

extern "C" {

size_t pc_prev_next_use_ws(uint64_t n) {
    size_t ctl;
    pc::sort_ctl(nullptr, n, &ctl);
    return ctl + pc::sort_bufs_bytes(n);
}

pc_status pc_prev_next_use(const uint64_t *keys, uint64_t n, uint32_t *prev, uint32_t *next,
                           const uint32_t *key_hist, void *ws, size_t ws_bytes, void *stream) {
    if (n >= (uint64_t)PC_NONE) return PC_ERR_TOO_LARGE;
    if (n > 0 && (!keys || !prev || !next)) return PC_ERR_INVALID;
    if (!ws) return PC_ERR_WORKSPACE;
    if (ws_bytes < pc_prev_next_use_ws(n)) return PC_ERR_WORKSPACE;
    hipStream_t s = (hipStream_t)stream;
    size_t ctl;
    const pc::SortCtl k = pc::sort_ctl(ws, n, &ctl);
    if (n == 0) return pc::fill_u32(reinterpret_cast<uint32_t *>(k.hdr), 0u, 1, s);
    return pc::prev_next_core(keys, n, nullptr, prev, next, key_hist, k, (char *)ws + ctl, s, nullptr,
                              pc::SortReport{});
}

}  // extern "C"
