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
// the digests are added to it.  Rounds pass through a ring of three LDS
// tiles (digests, turned into keys in place), and one barrier ends a phase.
// The chain wave also plans the rounds: it takes requests from a global
// counter, last to first (contexts grow turn by turn, so the longest chains
// start first), two rounds ahead of the digests, with the counter's answer
// and the request's table entries fetched while it chains.
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
constexpr int HASH_SWEEPS = 8;                                       // most sweeps (64 blocks) per digest wave and round
constexpr int HASH_ENTRIES = HASH_SWEEPS * DIGEST_WAVES * WAVE;      // most blocks per round: rows x SPAN
constexpr int HASH_RING = 4;                                         // token chunks in flight per digest wave
// Two workgroups per CU are enough to keep the vector units and the memory
// busy; with three or four the waves held each other up (on 2.2e8 accesses
// 2.62, 2.75 and 2.79 ms; with one 3.27; on 2.8e7, where the longest chain
// counts, 0.81, 0.97 and 1.16 ms).
constexpr int HASH_WG_PER_CU = 2;
static_assert(HASH_SWEEPS % HASH_RING == 0, "a round's chunks fill the ring a whole number of times");

// One row (request) of one round: its first token, the position of its first
// key, the number of blocks (0: none) and the first one's depth.
struct RoundRow {
    uint64_t tok;
    uint32_t pos, m, b;
};

template <int SPAN>
struct HashLds {
    static constexpr int ROWS = HASH_ENTRIES / SPAN;
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
        const uint32_t take = (uint32_t)lanes > 2 ? (uint32_t)lanes / 2 : 1u;
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
        constexpr int H = SPAN / WAVE;
        static_assert(DIGEST_WAVES % H == 0, "a wave's sweeps start at the same block of their rows");
        const int row0 = (w - 1) / H, first = (w - 1) % H * WAVE;   // sweep 0's row, and every sweep's first block
        RoundRow r2{}, r1{}, r0{}, rs{};   // rounds p + 2, p + 1, p, p - 1
        auto row_of = [&](int q) { return row0 + DIGEST_WAVES / H * q; };
        // blocks of sweep q (from 64 down; none below 1)
        auto count_of = [&](const RoundRow &r, int q) {
            return __builtin_amdgcn_readlane((int)r.m, row_of(q)) - first;
        };
        // Every lane loads, idle ones the sweep's first block or, without one,
        // a few unused header words: with a branch around a load the wait for
        // an older one would count as a wait for all.
        auto fetch = [&](TokChunk &c, const RoundRow &r, int q, int g) {
            const int cnt = count_of(r, q);
            const uint64_t tok = readlane64(r.tok, row_of(q)) + (uint64_t)(uint32_t)first * B + 16 * (uint32_t)g;
            const char *src = cnt > 0 ? reinterpret_cast<const char *>(tokens + tok)
                                      : reinterpret_cast<const char *>(idle);
            const uint32_t off = lane < cnt ? (uint32_t)lane * B * 4 : 0u;
            if (G16 == 1 || g < G - 1) load16(reinterpret_cast<const int32_t *>(src + off), c);
            else load_last(reinterpret_cast<const int32_t *>(src + off), last, c);
        };
        // sweep q's keys of round p - 1 leave the tile, and the digests of
        // round p + 1 take their place
        auto exchange = [&](uint64_t *tile, int q, int cnt, uint64_t d) {
            const int row = row_of(q);
            uint64_t *at = tile + row * ROW + lane;
            // (readlane before the branch: inside it a register may hold the
            // active lanes' values only)
            const int out = count_of(rs, q);
            const uint32_t pos = (uint32_t)__builtin_amdgcn_readlane((int)rs.pos, row);
            const uint32_t b = (uint32_t)__builtin_amdgcn_readlane((int)rs.b, row) + (uint32_t)first;
            const uint64_t o = deepest_first ? (uint64_t)pos - (uint32_t)first : (uint64_t)pos + (uint32_t)first;
            if (lane < out) {
                const uint64_t k = *at;
                const int64_t j = deepest_first ? -lane : lane;
                keys[o + j] = k;
                if (depth) depth[o + j] = b + (uint32_t)lane;
                if (key_hist) {
                    const uint32_t lo = (uint32_t)k;
#pragma unroll
                    for (int x = 0; x < 4; ++x) atomicAdd(&L.hist[256 * x + ((lo >> (8 * x)) & 0xFF)], 1u);
                }
            }
            if (lane < cnt) *at = d;
        };
        __syncthreads();   // phase -3: round 0 is planned
        if (lane < ROWS) r1 = L.rows[0][lane];
#pragma unroll
        for (int k = 0; k < HASH_RING; ++k) fetch(ring[k], r1, k / G, k % G);
        __syncthreads();   // phase -2
        for (int p = -1;; ++p) {
            // an opaque copy of the lane index: what is derived from it is worked
            // out where it is used, not kept (and spilled) across phases
            __asm__ volatile("" : "+v"(lane));
            if (lane < ROWS) r2 = L.rows[p & 1][lane];
            uint64_t *tile = L.tile[(p + 1) & 1] + first;
            if constexpr (G16 == 1) {
#pragma unroll
                for (int q = 0; q < HASH_SWEEPS; ++q) {
                    const int cnt = count_of(r1, q);
                    uint64_t d = 0;
                    if (cnt > 0) d = fold_end(fold16(0, ring[q % HASH_RING]));
                    exchange(tile, q, cnt, d);
                    if (q + HASH_RING < HASH_SWEEPS) fetch(ring[q % HASH_RING], r1, q + HASH_RING, 0);
                    else fetch(ring[q % HASH_RING], r2, q + HASH_RING - HASH_SWEEPS, 0);
                }
            } else {
                // chunk (q, g) is folded, chunk (fq, fg), four ahead, fetched;
                // past this round's chunks, the next round's first ones
                int q = 0, g = 0, fq = HASH_RING / G, fg = HASH_RING % G;
                uint64_t t = 0;
                while (q < sweeps) {
#pragma unroll
                    for (int k = 0; k < HASH_RING; ++k) {
                        const int cnt = count_of(r1, q);
                        if (cnt > 0) {
                            if (g < G - 1) t = fold16(t, ring[k]);
                            else t = fold_last(t, ring[k], last);
                        }
                        if (g == G - 1) {
                            exchange(tile, q, cnt, fold_end(t));
                            t = 0;
                        }
                        const bool here = fq < sweeps;
                        RoundRow from;
                        from.tok = here ? r1.tok : r2.tok;
                        from.m = here ? r1.m : r2.m;
                        fetch(ring[k], from, here ? fq : fq - sweeps, fg);
                        if (++g == G) { g = 0; ++q; }
                        if (++fg == G) { fg = 0; ++fq; }
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

}  // namespace pc

extern "C" {

size_t pc_hash_blocks_ws(uint32_t n_seqs) {
    (void)n_seqs;
    return pc::WS_HEADER + pc::WS_ALIGN;   // header + two work counters
}

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
    if (ws_bytes < pc_hash_blocks_ws(n_seqs)) return PC_ERR_WORKSPACE;
    hipStream_t s = (hipStream_t)stream;
    if (n_seqs == 0 || n_blocks == 0) {
        if (key_hist) return pc::fill_u32(key_hist, 0u, 4 * 256, s);
        return PC_OK;
    }
    pc::Carver c{(char *)ws, 0};
    int32_t *hdr = c.take<int32_t>(pc::WS_HEADER / sizeof(int32_t));
    uint32_t *counters = c.take<uint32_t>(2);
    pc::Fills fills;
    fills.add(hdr, 0u, 1);
    fills.add(counters, 0u, 2);
    if (key_hist) fills.add(key_hist, 0u, 4 * 256);
    const pc_status st = pc::fill_all(fills, s);
    if (st != PC_OK) return st;

    // Rows per workgroup: the requests spread over the resident workgroups.
    const uint64_t wgs = (uint64_t)pc::device_cus() * pc::HASH_WG_PER_CU;
    const uint64_t need = ((uint64_t)n_seqs + wgs - 1) / wgs;
    // Larger blocks take fewer rows: a digest wave folds at least eight chunks
    // of 16 tokens a phase (a multiple of the ring's four), and not many more,
    // so that the waves of a workgroup end their phases together (256-token
    // blocks, 1.7e6 accesses: 0.46 ms, with the eight sweeps of 16-token
    // blocks 0.85).
    const int chunks = ((int)block_size + 15) / 16;
    int sweeps = 1;
    while (sweeps < pc::HASH_SWEEPS && (sweeps * chunks < 8 || sweeps * chunks % pc::HASH_RING)) sweeps *= 2;
    // With few requests per workgroup a round takes more blocks of fewer rows:
    // what a phase costs besides the chain is then paid less often (17,758
    // requests, 35 per workgroup: 0.81 ms with 16 rows of 128 blocks, 0.84 with
    // 32 of 64, 0.92 with 8 of 256; 317 per workgroup: 2.64 and 2.59 ms).
    const uint64_t entries = (uint64_t)sweeps * pc::DIGEST_WAVES * pc::WAVE;
    const int span = need * 256 <= entries ? 256 : need * 32 <= entries ? 128 : 64;
    const int rows = (int)(entries / span);
    const int lanes = need < (uint64_t)rows ? (int)need : rows;
    const uint64_t want = ((uint64_t)n_seqs + lanes - 1) / lanes;
    const dim3 grid((unsigned)(want < wgs ? want : wgs));
    const dim3 block(pc::HASH_THREADS);
#define PC_HASH(S, G16)                                                                                              \
    PC_LAUNCH(pc::K_HASH, (pc::hash_kernel<S, G16>), grid, block, 0, s, tokens, n_tokens, tok_start, tok_len,        \
              n_seqs, block_size, parent, root, blk_off, n_blocks, keys, depth, key_hist, flags, counters, hdr, hdr + 16, lanes, sweeps)
    if (block_size == 16) {
        if (span == 256) PC_HASH(256, 1);
        else if (span == 128) PC_HASH(128, 1);
        else PC_HASH(64, 1);
    } else {
        if (span == 256) PC_HASH(256, 0);
        else if (span == 128) PC_HASH(128, 0);
        else PC_HASH(64, 0);
    }
#undef PC_HASH
    return PC_OK;
}

}  // extern "C"
