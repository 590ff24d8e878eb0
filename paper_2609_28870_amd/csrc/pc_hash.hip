// Chained block hashing (pc_hash_blocks).
//
// Block identity is a function of the whole token prefix (a KV state is
// reusable only if everything before it matches, Sec. 2.2); blocks are 16
// tokens (Sec. 3.1).  The hash is fixed in pc.h: splitmix64's finalizer used
// as a step S(x, w) = mix64((x ^ w) + gamma), folded over the block's
// token-pair words from 0 (the digest) and chained block to block.
//
// GPU mapping: one persistent kernel of specialised waves.  The chain is
// serial inside a request (one step is 20 instructions, 36 ns on one wave,
// whatever the number of lanes), the digests are independent, so a workgroup
// pairs one chain wave, a lane per request, with four digest waves, a lane
// per block, and runs them as a pipeline over rounds of SPAN blocks per
// request: while the chain wave walks round p, the digest waves load and fold
// the tokens of round p + 1 and write the keys of round p - 1 out, so a
// request advances at the chain's own pace and neither memory latency nor
// the digests are added to it.  Rounds pass through two LDS tiles in turn
// (digests, turned into keys in place), and one barrier ends a phase.  Round
// p + 1 goes to the tile that round p - 1 leaves in the same phase: a digest
// lane takes a key out of its place before it puts the digest there (exchange),
// and a place belongs to the same lane in every round.
// The chain wave also plans the rounds: it takes requests from a global
// counter, last to first (contexts grow turn by turn, so the longest chains
// come early; where it pays the requests are sorted by length first), two
// rounds ahead of the digests, with the counter's answer and the request's
// table entries fetched while it chains.
//
// Bound: the token reads where there are many requests (64 token bytes in
// and 8 key bytes out per 16-token block), the longest request's chain where
// there are few.  With a histogram pointer the kernel also counts the low
// four bytes of every key it writes (LDS, then one global add per bin), which
// the sort takes instead of a counting pass of its own.
#include "pc_internal.h"

namespace pc {

constexpr uint64_t GAMMA = 0x9E3779B97F4A7C15ull;

// mix64 without its last xor-shift (x ^ x >> 31), which the callers fold
// into the next step
__device__ __forceinline__ uint64_t mix64_open(uint64_t z) {
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    return (z ^ (z >> 27)) * 0x94D049BB133111EBull;
}

__device__ __forceinline__ uint64_t hstep(uint64_t x, uint64_t w) {
    const uint64_t t = mix64_open((x ^ w) + GAMMA);
    return t ^ (t >> 31);
}

// x ^ y ^ z, one three-input operation per half (gfx950 v_bitop3)
__device__ __forceinline__ uint64_t xor3(uint64_t x, uint64_t y, uint64_t z) {
    const uint32_t lo = __builtin_amdgcn_bitop3_b32((uint32_t)x, (uint32_t)y, (uint32_t)z, 0x96);
    const uint32_t hi = __builtin_amdgcn_bitop3_b32((uint32_t)(x >> 32), (uint32_t)(y >> 32), (uint32_t)(z >> 32), 0x96);
    return (uint64_t)lo | ((uint64_t)hi << 32);
}

// A digest in progress: t is the last step's value before its final xor-shift,
// which the next word's xor takes along (18 instead of 20 instructions a step).
// t = 0 stands for the start (0 ^ 0 >> 31 = 0).
__device__ __forceinline__ uint64_t fold(uint64_t t, uint32_t a, uint32_t b) {
    return mix64_open(xor3(t, t >> 31, (uint64_t)a | ((uint64_t)b << 32)) + GAMMA);
}
__device__ __forceinline__ uint64_t fold_end(uint64_t t) { return t ^ (t >> 31); }

// Token words at any 4-byte alignment: global loads of 16 bytes need no more
// on this part, so packed streams load as wide as aligned ones.
struct __attribute__((packed, aligned(4))) Tok4 {
    uint32_t x, y, z, w;
};
struct __attribute__((packed, aligned(4))) Tok2 {
    uint32_t x, y;
};

struct TokChunk {
    Tok4 v[4];
};
__device__ __forceinline__ void load16(const int32_t *p, TokChunk &c) {
    const Tok4 *q = reinterpret_cast<const Tok4 *>(p);
#pragma unroll
    for (int i = 0; i < 4; ++i) c.v[i] = q[i];
}
__device__ __forceinline__ uint64_t fold16(uint64_t t, const TokChunk &c) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        t = fold(t, c.v[i].x, c.v[i].y);
        t = fold(t, c.v[i].z, c.v[i].w);
    }
    return t;
}
// a chunk of `count` tokens (even, 2 .. 16)
__device__ __forceinline__ void load_last(const int32_t *p, int count, TokChunk &c) {
    if (count == 16) return load16(p, c);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (4 * i + 4 <= count) {
            c.v[i] = reinterpret_cast<const Tok4 *>(p)[i];
        } else if (4 * i + 2 <= count) {
            const Tok2 x = reinterpret_cast<const Tok2 *>(p)[2 * i];
            c.v[i].x = x.x;
            c.v[i].y = x.y;
        }
    }
}
__device__ __forceinline__ uint64_t fold_last(uint64_t t, const TokChunk &c, int count) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (4 * i + 2 <= count) t = fold(t, c.v[i].x, c.v[i].y);
        if (4 * i + 4 <= count) t = fold(t, c.v[i].z, c.v[i].w);
    }
    return t;
}

// true when every token and block of request r lies inside the arrays
__device__ __forceinline__ bool request_in_bounds(uint64_t st, uint32_t len, uint32_t nb, uint64_t out,
                                                  uint64_t n_tokens, uint64_t n_blocks) {
    return st <= n_tokens && len <= n_tokens - st && out <= n_blocks && nb <= n_blocks - out;
}

constexpr int DIGEST_WAVES = 4;
constexpr int HASH_THREADS = (1 + DIGEST_WAVES) * WAVE;
constexpr int HASH_SWEEPS = 8;                                      // most sweeps (64 blocks) per digest wave and round
constexpr int HASH_ENTRIES = HASH_SWEEPS * DIGEST_WAVES * WAVE;     // most blocks per round: rows x SPAN
constexpr int HASH_RING = 4;                                        // token chunks in flight per digest wave
// At most two workgroups per CU: they keep the vector units and the memory
// busy; with three or four the waves held each other up (on 2.2e8 accesses
// 2.10 ms, with three 2.35; on 2.8e7, where the longest chain counts, 0.66 and
// 0.83 ms).
constexpr int HASH_WG_PER_CU = 2;

// One row (request) of one round: its first token, the position of its first
// key, the number of blocks (0: none) and the first one's depth.
struct RoundRow {
    uint64_t tok;
    uint32_t pos, m, b;
};

template <int SPAN>
struct HashLds {
    static constexpr int ROWS = HASH_ENTRIES / SPAN < WAVE ? HASH_ENTRIES / SPAN : WAVE;
    static constexpr int ROW = SPAN + 1;         // padded: a lane per row reads without bank conflicts
    uint64_t tile[2][ROWS * ROW];                // round r in tile r mod 2
    RoundRow rows[2][ROWS];                      // round r in rows[r mod 2]
    uint32_t hist[4 * 256];                      // byte histograms of the keys written
    int32_t end;                                 // first round with no work from there on
};

// the chain over `steps` entries (a multiple of 16) of one row: while eight
// are walked the next eight are read from LDS
__device__ __forceinline__ uint64_t chain_row(uint64_t key, uint64_t *row, int steps) {
    uint64_t d[8], e[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) d[k] = row[k];
    for (int q = 0; q < steps; q += 16) {
#pragma unroll
        for (int k = 0; k < 8; ++k) e[k] = row[q + 8 + k];
#pragma unroll
        for (int k = 0; k < 8; ++k) row[q + k] = key = hstep(key, d[k]);
        const int nx = q + 16 < steps ? q + 16 : q;
#pragma unroll
        for (int k = 0; k < 8; ++k) d[k] = row[nx + k];
#pragma unroll
        for (int k = 0; k < 8; ++k) row[q + 8 + k] = key = hstep(key, e[k]);
    }
    return key;
}

// G16: chunks of 16 tokens per block when known at compile time (1 for
// 16-token blocks), 0 for any block size
template <int SPAN, int G16>
__global__ __launch_bounds__(HASH_THREADS, 4) void hash_kernel(
    const int32_t *__restrict__ tokens, uint64_t n_tokens, const uint64_t *__restrict__ tok_start,
    const uint32_t *__restrict__ tok_len, uint32_t n_seqs, uint32_t B, const uint64_t *__restrict__ parent,
    uint64_t root, const uint64_t *__restrict__ blk_off, uint64_t n_blocks, uint64_t *__restrict__ keys,
    uint32_t *__restrict__ depth, uint32_t *__restrict__ key_hist, uint32_t flags, uint32_t *__restrict__ counter,
    int32_t *__restrict__ err, const int32_t *__restrict__ idle, int lanes, int sweeps) {
    using Lds = HashLds<SPAN>;
    constexpr int ROWS = Lds::ROWS, ROW = Lds::ROW;
    __shared__ Lds L;
    const bool deepest_first = (flags & PC_HASH_DEEPEST_FIRST) != 0;
    int lane = threadIdx.x & (WAVE - 1);
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / WAVE));
    for (int i = threadIdx.x; i < 4 * 256; i += HASH_THREADS) L.hist[i] = 0;
    if (threadIdx.x == 0) L.end = 0x7FFFFFFF;
    __syncthreads();

    // Phase p: chain round p, digest round p + 1, load round p + 2, plan round
    // p + 3, store round p - 1.  Both kinds of waves pass one barrier a phase.
    if (w == 0) {
        __builtin_amdgcn_s_setprio(2);   // every phase waits for the chain
        // The row's request (nb blocks, the next round to plan starts at block
        // b), the one to follow (`ahead`: its table entries are on the way),
        // and what the chain needs of the rounds planned (m entries; whether
        // the round starts a request, and its key).
        bool busy = false, ahead = false;
        uint32_t nb = 0, b = 0;
        uint64_t st = 0, out = 0, start_key = 0;
        uint32_t n_len = 0;
        uint64_t n_st = 0, n_out = 0, n_key = 0;
        uint32_t m0 = 0, m1 = 0, m2 = 0;
        bool new0 = false, new1 = false, new2 = false;
        uint64_t key = 0, init0 = 0, init1 = 0, init2 = 0;
        // Requests not begun yet (wave-uniform): the first ones are dealt out
        // without the counter, neighbours (often equally long) to different
        // workgroups; later ones are taken `take` at a time.
        const uint32_t dealt = gridDim.x * (uint32_t)lanes;
        // (short requests: a row may need one each round)
        const bool brief = n_blocks / n_seqs < (uint64_t)SPAN;
        const uint32_t take = brief || lanes < 2 ? (uint32_t)lanes : (uint32_t)lanes / 2;
        uint32_t pool = 0, pool_end = 0;      // counter range in hand
        bool asking = false, exhausted = dealt >= n_seqs;
        uint32_t asked = 0;
        for (int p = -3;; ++p) {
            if (pool == pool_end && asking) {
                pool = dealt + (uint32_t)__builtin_amdgcn_readfirstlane((int)asked);
                pool = pool < n_seqs ? pool : n_seqs;
                pool_end = n_seqs - pool < take ? n_seqs : pool + take;
                asking = false;
                exhausted = pool_end == n_seqs;   // the counter only grows
            }
            // rows that end within two rounds get the request to follow
            const bool want = !ahead && lane < lanes && (!busy || nb - b <= 2 * SPAN);
            uint32_t taken = n_seqs;
            if (p == -3) {
                taken = lane < lanes ? (uint32_t)lane * gridDim.x + blockIdx.x : n_seqs;
                taken = taken < n_seqs ? taken : n_seqs;
            } else {
                const uint64_t wm = ballot(want);
                const uint32_t left = pool_end - pool, nw = (uint32_t)__popcll(wm);
                if (want && mbcnt(wm) < left) taken = pool + mbcnt(wm);
                pool += nw < left ? nw : left;
            }
            if (taken < n_seqs) {
                const uint32_t r = n_seqs - 1 - taken;
                n_len = tok_len[r];
                n_st = tok_start[r];
                n_out = blk_off[r];
                n_key = parent ? parent[r] : root;
                ahead = true;
            }
            if (!asking && !exhausted && pool_end - pool <= take / 2) {
                // (a per-lane address: the compiler would wait at once for the
                // answer of an atomic on a uniform one)
                uint32_t *c = counter;
                __asm__ volatile("" : "+v"(c));
                if (lane == 0) asked = atomicAdd(c, take);
                asking = true;
            }
            // The chain of round p.  Every row walks as far as the longest one:
            // only a request's last round is short, and what lies past its end
            // is neither stored nor carried on.
            const uint32_t longest = (uint32_t)__builtin_amdgcn_readlane((int)wave_incl_max(m0), WAVE - 1);
            if (longest) {
                if (lane < ROWS)
                    key = chain_row(new0 ? init0 : key, L.tile[p & 1] + lane * ROW, (int)((longest + 15) & ~15u));
            }
            // plan round p + 3
            if (!busy && ahead) {
                ahead = false;
                nb = n_len / B;
                st = n_st;
                out = n_out;
                b = 0;
                start_key = n_key;
                if (request_in_bounds(st, n_len, nb, out, n_tokens, n_blocks))
                    busy = nb > 0;
                else
                    atomicOr(err, DEV_ERR_BAD_LAYOUT);
            }
            m0 = m1;
            new0 = new1;
            init0 = init1;
            m1 = m2;
            new1 = new2;
            init1 = init2;
            m2 = busy ? (nb - b < (uint32_t)SPAN ? nb - b : (uint32_t)SPAN) : 0u;
            new2 = b == 0;
            init2 = start_key;
            if (lane < ROWS)
                L.rows[(p + 3) & 1][lane] = RoundRow{
                    st + (uint64_t)b * B, (uint32_t)(deepest_first ? out + nb - 1 - b : out + b), m2, b};
            b += m2;
            busy = busy && b < nb;
            if (ballot(m2 != 0 || busy || ahead) == 0 && exhausted && pool == pool_end && lane == 0 && L.end > p + 3)
                L.end = p + 3;
            __syncthreads();
            if (p >= L.end) break;
        }
    } else {
        // A sweep is 64 blocks of one row; this wave takes sweeps w - 1 +
        // DIGEST_WAVES q.  Lane r holds row r of the rounds in work (its
        // values reach the wave by readlane, so addresses are scalar).  A
        // block's tokens come in chunks of 16; the chunks of the wave's
        // sweeps, sweep by sweep, pass through a ring of register buffers, so
        // that four are always on their way, the next round's first ones
        // across the barrier.
        const int G = G16 ? G16 : (int)((B + 15) / 16);
        const int last = G16 ? 16 : (int)(B - 16 * (uint32_t)(G - 1));   // tokens of a block's last chunk
        TokChunk ring[HASH_RING];
        // (spans under 64: a sweep is the blocks of 64 / SPAN rows, and each
        // lane fetches its row's values by ds_bpermute)
        constexpr bool SHORT = SPAN < WAVE;
        constexpr int H = SHORT ? 1 : SPAN / WAVE, RPS = SHORT ? WAVE / SPAN : 1;
        constexpr int SWEEPS = ROWS * SPAN / (DIGEST_WAVES * WAVE);   // of 16-token blocks
        static_assert(SWEEPS % HASH_RING == 0, "a round's chunks fill the ring a whole number of times");
        static_assert(DIGEST_WAVES % H == 0, "a wave's sweeps start at the same block of their rows");
        // sweep 0's (first) row, and every sweep's first block
        const int row0 = (w - 1) / H * RPS, first = (w - 1) % H * WAVE;
        RoundRow r2{}, r1{}, r0{}, rs{};   // rounds p + 2, p + 1, p, p - 1
        auto row_of = [&](int q) { return row0 + DIGEST_WAVES / H * RPS * q; };
        // blocks of the sweep at `row` (from 64 down; none below 1)
        auto count_of = [&](const RoundRow &r, int row) { return __builtin_amdgcn_readlane((int)r.m, row) - first; };
        // SHORT: value x of the row that this lane's block is in
        auto of_row = [&](uint32_t x, int row) {
            return (uint32_t)__builtin_amdgcn_ds_bpermute(4 * (row + lane / SPAN), (int)x);
        };
        // Every lane loads, idle ones the sweep's first block or, without one,
        // a few unused header words: with a branch around a load the wait for
        // an older one would count as a wait for all.
        auto fetch = [&](TokChunk &c, const RoundRow &r, int row, bool any, int g) {
            if constexpr (SHORT) {
                const uint32_t sub = lane % SPAN;
                const bool mine = any && sub < of_row(r.m, row);
                const uint64_t tok = (uint64_t)of_row((uint32_t)r.tok, row) |
                                     (uint64_t)of_row((uint32_t)(r.tok >> 32), row) << 32;
                const int32_t *src = mine ? tokens + tok + sub * B + 16 * (uint32_t)g : idle;
                if (g < G - 1) load16(src, c);
                else load_last(src, last, c);
                return;
            }
            const int cnt = any ? count_of(r, row) : 0;
            const uint64_t tok = readlane64(r.tok, row) + (uint64_t)(uint32_t)first * B + 16 * (uint32_t)g;
            const char *src = cnt > 0 ? reinterpret_cast<const char *>(tokens + tok)
                                      : reinterpret_cast<const char *>(idle);
            const uint32_t off = lane < cnt ? (uint32_t)lane * B * 4 : 0u;
            if (G16 == 1 || g < G - 1) load16(reinterpret_cast<const int32_t *>(src + off), c);
            else load_last(reinterpret_cast<const int32_t *>(src + off), last, c);
        };
        // the sweep's keys of round p - 1 leave the tile, and the digests of
        // round p + 1 take their place
        auto put = [&](uint64_t k, uint64_t at, uint32_t b) {
            keys[at] = k;
            if (depth) depth[at] = b;
            if (key_hist) {
                const uint32_t lo = (uint32_t)k;
#pragma unroll
                for (int x = 0; x < 4; ++x) atomicAdd(&L.hist[256 * x + ((lo >> (8 * x)) & 0xFF)], 1u);
            }
        };
        auto exchange = [&](uint64_t *tile, int row, int cnt, uint64_t d) {
            if constexpr (SHORT) {
                const uint32_t sub = lane % SPAN, out = of_row(rs.m, row), pos = of_row(rs.pos, row);
                const uint32_t b = of_row(rs.b, row), in = of_row(r1.m, row);
                uint64_t *at = tile + (row + lane / SPAN) * ROW + sub;
                if (sub < out) put(*at, deepest_first ? pos - sub : pos + sub, b + sub);
                if (sub < in) *at = d;
                return;
            }
            uint64_t *at = tile + row * ROW + lane;
            // (readlane before the branch: inside it a register may hold the
            // active lanes' values only)
            const int out = count_of(rs, row);
            const uint32_t pos = (uint32_t)__builtin_amdgcn_readlane((int)rs.pos, row);
            const uint32_t b = (uint32_t)__builtin_amdgcn_readlane((int)rs.b, row) + (uint32_t)first;
            const uint64_t o = deepest_first ? (uint64_t)pos - (uint32_t)first : (uint64_t)pos + (uint32_t)first;
            if (lane < out) {
                const int64_t j = deepest_first ? -lane : lane;
                put(*at, o + j, b + (uint32_t)lane);
            }
            if (lane < cnt) *at = d;
        };
        // this wave's sweeps that have blocks in a round, as a mask of their
        // (first) rows
        uint64_t mine = 0;
        for (int q = 0; G16 != 1 && q < sweeps; ++q) mine |= 1ull << row_of(q);
        auto sweeps_in = [&](const RoundRow &r) {
            uint64_t m = ballot(r.m > (uint32_t)first);
            if constexpr (SHORT)
                for (int x = 1; x < RPS; x *= 2) m |= m >> x;
            return m & mine;
        };
        // the chunks to fetch, a sweep after the other: the sweeps left and the
        // next one's next chunk (none left: an idle fetch)
        uint64_t left = 0;
        int chunk = 0;
        auto fetch_next = [&](TokChunk &c, const RoundRow &r) {
            fetch(c, r, left ? __builtin_ctzll(left) : 0, left != 0, chunk);
            if (left && ++chunk == G) {
                chunk = 0;
                left &= left - 1;
            }
        };
        __syncthreads();   // phase -3: round 0 is planned
        if (lane < ROWS) r1 = L.rows[0][lane];
        if (G16 != 1) left = sweeps_in(r1);
#pragma unroll
        for (int k = 0; k < HASH_RING; ++k) {
            if constexpr (G16 == 1) fetch(ring[k], r1, row_of(k), true, 0);
            else fetch_next(ring[k], r1);
        }
        __syncthreads();   // phase -2
        for (int p = -1;; ++p) {
            // an opaque copy of the lane index: what is derived from it is worked
            // out where it is used, not kept (and spilled) across phases
            __asm__ volatile("" : "+v"(lane));
            if (lane < ROWS) r2 = L.rows[p & 1][lane];
            uint64_t *tile = L.tile[(p + 1) & 1] + first;
            if constexpr (G16 == 1) {
#pragma unroll
                for (int q = 0; q < SWEEPS; ++q) {
                    const int row = row_of(q);
                    const int cnt = SHORT ? __popcll(ballot((uint32_t)(lane % SPAN) < of_row(r1.m, row))) : count_of(r1, row);
                    uint64_t d = 0;
                    if (cnt > 0) d = fold_end(fold16(0, ring[q % HASH_RING]));
                    exchange(tile, row, cnt, d);
                    if (q + HASH_RING < SWEEPS) fetch(ring[q % HASH_RING], r1, row_of(q + HASH_RING), true, 0);
                    else fetch(ring[q % HASH_RING], r2, row_of(q + HASH_RING - SWEEPS), true, 0);
                }
            } else {
                // Sweeps without blocks are passed over, so that a round costs
                // what it holds: the ones that only have keys to store first.
                uint64_t now = sweeps_in(r1);
                for (uint64_t out = sweeps_in(rs) & ~now; out; out &= out - 1) exchange(tile, __builtin_ctzll(out), 0, 0);
                // A chunk is folded, the one four ahead fetched; past this round's
                // chunks (rounded up to fours, at least four), the next round's
                // first ones.
                int quads = (__popcll(now) * G + HASH_RING - 1) / HASH_RING, g = 0;
                quads = quads ? quads : 1;
                uint64_t t = 0;
                for (; quads; --quads) {
                    const bool here = quads > 1;
                    if (!here) {
                        left = sweeps_in(r2);
                        chunk = 0;
                    }
#pragma unroll
                    for (int k = 0; k < HASH_RING; ++k) {
                        if (now) {
                            if (g < G - 1) t = fold16(t, ring[k]);
                            else t = fold_last(t, ring[k], last);
                            if (++g == G) {
                                const int row = __builtin_ctzll(now);
                                exchange(tile, row, SHORT ? WAVE : count_of(r1, row), fold_end(t));
                                t = 0;
                                g = 0;
                                now &= now - 1;
                            }
                        }
                        // two at a time: mostly the halves of the same lines,
                        // which do not stay in the caches until the next fetch
                        if (k % 2)
#pragma unroll
                            for (int x = k - 1; x <= k; ++x) {
                                RoundRow from;
                                from.tok = here ? r1.tok : r2.tok;
                                from.m = here ? r1.m : r2.m;
                                fetch_next(ring[x], from);
                            }
                    }
                }
            }
            rs = r0;
            r0 = r1;
            r1 = r2;
            __syncthreads();
            if (p >= L.end) break;
        }
    }
    if (key_hist) {
        for (int i = threadIdx.x; i < 4 * 256; i += HASH_THREADS)
            if (L.hist[i]) atomicAdd(&key_hist[i], L.hist[i]);
    }
}

// ---- requests in the order of their length -------------------------------
// The last request to end decides the kernel's time, so the longest should
// start first.  A counting sort over 1024 length classes (32 to an octave, 3%
// apart) copies the requests' table entries into that order: the hash kernel
// walks them instead of the caller's, last to first as before.
constexpr int LEN_CLASSES = 1024, ORDER_THREADS = 256;
// requests: fewer are all in work at once, and among more the last hardly counts
constexpr uint32_t ORDER_MIN = 1u << 10, ORDER_MAX = 1u << 24;
__device__ __forceinline__ int length_class(uint32_t len, uint32_t B) {
    const uint32_t nb = len / B;
    if (nb < 32) return (int)nb;
    const int e = 26 - __clz((int)nb);   // the five bits below the leading one
    return 32 + e * 32 + (int)((nb >> e) & 31);
}

struct OrderWs {
    uint32_t *hist, *ticket;   // hist[LEN_CLASSES], ticket: zeroed before
    uint32_t *cursor;          // [LEN_CLASSES]
    uint64_t *start, *off, *parent;
    uint32_t *len;
};

// counts the classes; the last workgroup turns them into first positions
__global__ __launch_bounds__(ORDER_THREADS) void hash_classes_kernel(const uint32_t *__restrict__ tok_len, uint32_t n,
                                                                     uint32_t B, OrderWs o) {
    __shared__ uint32_t h[LEN_CLASSES], tmp[ORDER_THREADS / WAVE], mine;
    for (int i = threadIdx.x; i < LEN_CLASSES; i += ORDER_THREADS) h[i] = 0;
    __syncthreads();
    for (uint32_t i = blockIdx.x * ORDER_THREADS + threadIdx.x; i < n; i += gridDim.x * ORDER_THREADS)
        atomicAdd(&h[length_class(tok_len[i], B)], 1u);
    __syncthreads();
    for (int i = threadIdx.x; i < LEN_CLASSES; i += ORDER_THREADS)
        if (h[i]) atomicAdd(&o.hist[i], h[i]);
    atomics_performed();
    __syncthreads();
    if (threadIdx.x == 0) mine = atomicAdd(o.ticket, 1u);
    __syncthreads();
    if (mine != gridDim.x - 1) return;
    constexpr int PER = LEN_CLASSES / ORDER_THREADS;
    uint32_t v[PER], sum = 0, total;
    for (int k = 0; k < PER; ++k) sum += v[k] = ld_status(&o.hist[threadIdx.x * PER + k]);
    uint32_t at = block_excl_scan(sum, tmp, &total);
    for (int k = 0; k < PER; ++k) {
        o.cursor[threadIdx.x * PER + k] = at;
        at += v[k];
    }
}

// each workgroup takes room for its chunk's classes and moves the entries
__global__ __launch_bounds__(ORDER_THREADS) void hash_order_kernel(
    const uint64_t *__restrict__ tok_start, const uint32_t *__restrict__ tok_len,
    const uint64_t *__restrict__ blk_off, const uint64_t *__restrict__ parent, uint32_t n, uint32_t B, uint32_t per,
    OrderWs o) {
    __shared__ uint32_t h[LEN_CLASSES];
    const uint32_t lo = blockIdx.x * per, hi = n - lo < per ? n : lo + per;
    for (int i = threadIdx.x; i < LEN_CLASSES; i += ORDER_THREADS) h[i] = 0;
    __syncthreads();
    for (uint32_t i = lo + threadIdx.x; i < hi; i += ORDER_THREADS) atomicAdd(&h[length_class(tok_len[i], B)], 1u);
    __syncthreads();
    for (int i = threadIdx.x; i < LEN_CLASSES; i += ORDER_THREADS)
        if (h[i]) h[i] = atomicAdd(&o.cursor[i], h[i]);
    __syncthreads();
    for (uint32_t i = lo + threadIdx.x; i < hi; i += ORDER_THREADS) {
        const uint32_t len = tok_len[i];
        const uint32_t at = atomicAdd(&h[length_class(len, B)], 1u);
        o.len[at] = len;
        o.start[at] = tok_start[i];
        o.off[at] = blk_off[i];
        if (parent) o.parent[at] = parent[i];
    }
}

// the workspace: header, work counters, then what the order needs
struct HashWs {
    int32_t *hdr;
    uint32_t *counters;
    OrderWs order;
    size_t least, bytes;   // without and with the order
};
static HashWs hash_ws(void *ws, uint32_t n_seqs) {
    Carver c{(char *)ws, 0};
    HashWs w;
    w.hdr = c.take<int32_t>(WS_HEADER / sizeof(int32_t));
    w.counters = c.take<uint32_t>(3);
    w.order.ticket = w.counters + 2;
    w.least = WS_HEADER + WS_ALIGN;
    w.bytes = w.least;
    if (n_seqs <= ORDER_MIN || n_seqs > ORDER_MAX) return w;
    w.order.hist = c.take<uint32_t>(LEN_CLASSES);
    w.order.cursor = c.take<uint32_t>(LEN_CLASSES);
    w.order.start = c.take<uint64_t>(n_seqs);
    w.order.off = c.take<uint64_t>(n_seqs);
    w.order.parent = c.take<uint64_t>(n_seqs);
    w.order.len = c.take<uint32_t>(n_seqs);
    w.bytes = c.off;
    return w;
}

}  // namespace pc

extern "C" {

size_t pc_hash_blocks_ws(uint32_t n_seqs) { return pc::hash_ws(nullptr, n_seqs).bytes; }

pc_status pc_hash_blocks(const int32_t *tokens, uint64_t n_tokens, const uint64_t *tok_start,
                         const uint32_t *tok_len,
                         uint32_t n_seqs, uint32_t block_size, const uint64_t *parent, uint64_t root,
                         const uint64_t *blk_off, uint64_t n_blocks, uint64_t *keys, uint32_t *depth,
                         uint32_t *key_hist, uint32_t flags, void *ws, size_t ws_bytes, void *stream) {
    if (block_size < 2 || block_size > 1024 || (block_size & 1)) return PC_ERR_INVALID;
    if (n_seqs >= 0x80000000u) return PC_ERR_TOO_LARGE;
    if (n_blocks >= (uint64_t)PC_NONE) return PC_ERR_TOO_LARGE;
    if (n_seqs > 0 && (!tokens || !tok_start || !tok_len || !blk_off)) return PC_ERR_INVALID;
    if (n_blocks > 0 && !keys) return PC_ERR_INVALID;
    if (!ws) return PC_ERR_WORKSPACE;
    const pc::HashWs hw = pc::hash_ws(ws, n_seqs);
    if (ws_bytes < hw.least) return PC_ERR_WORKSPACE;
    hipStream_t s = (hipStream_t)stream;
    if (n_seqs == 0 || n_blocks == 0) {
        if (key_hist) return pc::fill_u32(key_hist, 0u, 4 * 256, s);
        return PC_OK;
    }
    // Larger blocks take fewer rows: a digest wave folds at least sixteen chunks
    // of 16 tokens a phase (a multiple of the ring's four), and not many more,
    // so that the waves of a workgroup end their phases together (64-token
    // blocks, 5.0e7 accesses: 2.12 ms, with eight chunks 2.28; 256-token blocks,
    // 1.7e6: 0.46 ms, with the eight sweeps of 16-token blocks 0.85).
    const int chunks = ((int)block_size + 15) / 16;
    int sweeps = 1;
    while (sweeps < pc::HASH_SWEEPS && (sweeps * chunks < 16 || sweeps * chunks % pc::HASH_RING)) sweeps *= 2;
    const uint64_t cus = (uint64_t)pc::device_cus(), mean = n_blocks / n_seqs;
    const uint64_t need = (n_seqs + 2 * cus - 1) / (2 * cus);
    int per_cu = pc::HASH_WG_PER_CU, span = 0;
    // Many short requests: a round of 64 blocks of one request would leave most
    // of it empty, so a sweep takes blocks of several requests.  The few long
    // ones that may be among them pay for the shorter rounds, hence not for
    // fewer requests (us with spans of 16 / 32 / 64 and, in brackets, of a wave
    // per 64 requests that walks them 32 blocks at a time):
    //   16 tokens, 1.0e6 requests of 1..8 blocks    208 239 419 (388)
    //              1.0e6 of 1..32                   407 267 479 (447)
    //              1.0e5 of 13, log-normal          244 237 200 (451)
    //   32 tokens, 1.0e6 of 1..8                    308 541 974 (580)
    //              1.0e4 of 1..32                    26  25  39  (45)
    //   64 tokens, 5.0e5 of 1..8                    274 496 898 (491)
    //              5.0e5 of 1..32                   651 706 1010 (621)
    //              1.0e4 of 26, log-normal          380 209 182 (366)
    if (chunks < 8) {
        const bool few_tokens = block_size < 16, one = block_size == 16;
        const uint32_t many = one ? 1u << 19 : chunks == 2 || chunks == 3 ? 1u << 13 : 1u << 16;
        if (mean < 12 && n_seqs >= 1u << 19 && chunks > 1) span = 16;
        else if (mean < (few_tokens ? 128 : 48) && n_seqs >= many) span = 32;
        else if (mean < 24 && n_seqs >= 1u << 11 && !one) span = 64;
    }
    const uint64_t sweep = pc::DIGEST_WAVES * pc::WAVE;   // blocks of one sweep of every digest wave
    while (span && sweeps * sweep / span > pc::WAVE) sweeps /= 2;   // a lane of the chain wave per row
    // Rows in work at once (256 CUs x workgroups per CU x entries / span): the
    // fewer, the closer each request runs to its chain's own pace; the more,
    // the better the memory is used.  Best is about a quarter of the requests,
    // so that the shorter ones fill up behind the longest.  16-token blocks,
    // ms with 16384 / 8192 / 4096 / 2048 rows:
    //   156,497 requests of 1433 blocks on average  2.00 2.57 2.64 3.97
    //    42,000                         1433        0.92 0.83 0.99 1.55
    //    17,233                         1604        0.68 0.66 0.52 0.72
    //     8,700                         1604        0.49 0.48 0.45 0.41
    //    11,700                          171        0.12 0.13 0.13 0.20
    // Larger blocks have more tokens to a chain step and fewer rows: they keep
    // two workgroups per CU.  From 128 tokens on, where a request has few
    // blocks, a sweep of 64 takes them from several rows, or its lanes would
    // idle (ms with spans of 16 / 32 / 64 / 128: 2.0e7 blocks of 128 tokens in
    // 111,000 requests 1.60 1.63 1.72 2.08; 1.0e7 of 256 in 111,000 1.54 1.68
    // 2.16 2.26; 1.7e6 of 256 in 18,389 0.44 0.32 0.38 0.41; with smaller
    // blocks the shorter rounds cost more: 5.0e7 of 64 in 156,000 2.77 against
    // 2.01).
    const uint64_t entries = sweeps * sweep;
    for (int x = chunks < 8 ? 64 : 16; x <= 128 && !span; x *= 2)
        if (entries / x <= pc::WAVE && n_seqs >= 4 * per_cu * cus * (entries / x)) span = x;
    if (!span && sweeps == pc::HASH_SWEEPS) {
        per_cu = 1;
        const uint64_t r = cus * (entries / 256);
        span = n_seqs <= r || (mean >= 512 && n_seqs <= 6 * r) ? 256 : 128;
    } else if (!span) {
        span = need * 256 <= entries ? 256 : need * 32 <= entries ? 128 : 64;
    }
    if (chunks >= 8 && mean < 48) {
        // (8192 requests of 8 blocks of 128 tokens 0.078 ms, with 64 0.094)
        if (span == 64 && mean < 32 && n_seqs >= 8 * cus * (entries / 128)) span = 32;
        // with more than a few blocks to a request they differ in length, and the
        // long ones pay (1.0e5 of 13 blocks of 256 tokens, log-normal, us with 16
        // / 32 / 64: 1908 1071 740; of 27 3216 1811 1073; 1..32 530 524 737)
        if (span == 16 && mean >= 12) span = 32;
        if (span == 32 && mean >= 24 && chunks >= 16) span = 64;
        // (1.0e4 requests of 1..32 blocks of 128 tokens 66 us, with 128 81)
        if (span == 128 && mean < 24 && n_seqs >= 1u << 13 && chunks < 16) span = 64;
    }
    const uint64_t wgs = cus * per_cu, most = ((uint64_t)n_seqs + wgs - 1) / wgs;
    const int rows = (int)(entries / span);
    const int lanes = most < (uint64_t)rows ? (int)most : rows;
    const uint64_t want = ((uint64_t)n_seqs + lanes - 1) / lanes;
    const dim3 grid((unsigned)(want < wgs ? want : wgs));
    const dim3 block(pc::HASH_THREADS);
    // The order pays where requests are still waiting when the first ones end
    // and the work is long against the two launches (12 us): 2.8e7 accesses
    // 0.80 -> 0.66 ms, 2.2e8 2.71 -> 2.05, 8.0e8 7.90 -> 7.44.
    const bool ordered = hw.bytes > hw.least && n_seqs > grid.x * (uint64_t)lanes && mean * block_size >= 1024 &&
                         n_blocks * block_size >= 1ull << 26 && ws_bytes >= hw.bytes;
    pc::Fills fills;
    fills.add(hw.hdr, 0u, 1);
    fills.add(hw.counters, 0u, 3);
    if (ordered) fills.add(hw.order.hist, 0u, pc::LEN_CLASSES);
    if (key_hist) fills.add(key_hist, 0u, 4 * 256);
    const pc_status st = pc::fill_all(fills, s);
    if (st != PC_OK) return st;
    if (ordered) {
        const uint32_t T = pc::ORDER_THREADS;
        const uint32_t groups = n_seqs / (4 * T) < 256 ? n_seqs / (4 * T) + 1 : 256;
        const uint32_t per = (n_seqs + groups - 1) / groups;
        PC_LAUNCH(pc::K_HASH_ORDER, pc::hash_classes_kernel, dim3(groups), dim3(T), 0, s, tok_len, n_seqs, block_size,
                  hw.order);
        PC_LAUNCH(pc::K_HASH_ORDER, pc::hash_order_kernel, dim3((n_seqs + per - 1) / per), dim3(T), 0, s, tok_start,
                  tok_len, blk_off, parent, n_seqs, block_size, per, hw.order);
        tok_start = hw.order.start;
        tok_len = hw.order.len;
        blk_off = hw.order.off;
        if (parent) parent = hw.order.parent;
    }
#define PC_HASH(S, G16)                                                                                              \
    PC_LAUNCH(pc::K_HASH, (pc::hash_kernel<S, G16>), grid, block, 0, s, tokens, n_tokens, tok_start, tok_len,        \
              n_seqs, block_size, parent, root, blk_off, n_blocks, keys, depth, key_hist, flags, hw.counters,       \
              hw.hdr, hw.hdr + 16, lanes, sweeps)
    if (block_size == 16) {
        if (span == 256) PC_HASH(256, 1);
        else if (span == 128) PC_HASH(128, 1);
        else if (span == 64) PC_HASH(64, 1);
        else PC_HASH(32, 1);
    } else {
        if (span == 256) PC_HASH(256, 0);
        else if (span == 128) PC_HASH(128, 0);
        else if (span == 64) PC_HASH(64, 0);
        else if (span == 32) PC_HASH(32, 0);
        else PC_HASH(16, 0);
    }
#undef PC_HASH
    return PC_OK;
}

}  // extern "C"
