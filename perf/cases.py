"""Workloads the library's speed is measured on.

Every case is a call (or the sequence of calls) that a program scoring
prefix-cache eviction makes through ``paper_2609_28870_amd.pc``: request logs
through ``Pipeline`` in its three residency modes and through ``Profiler``,
key streams through the generic stages, Belady's MIN, and block hashing for a
batch of turns.  Sizes run from one scheduler step to 8e8 block accesses.

Request logs are windows of exactly ``accesses`` block accesses of a session
process with the shapes the repository's traces have (append-only turns that
re-send the whole context, heavy-tailed turn counts and lengths, shared system
prompts, Poisson session starts); the last request of the window is cut to
fit.  All outputs are integers with one right value, so they compare exactly.
"""
import math

import numpy as np
import torch

from paper_2609_28870_amd import pc

VOCAB = 151936
SYS_LEN, SYS_PROMPTS = 2048, 32
NONE = 0xFFFFFFFF
GOLDEN = 0x9E3779B97F4A7C15
ALPHA_PER_TOKEN = 2 * 3_000_000_000     # recompute cost of a block at depth d: alpha + beta d
TABLE_BLOCKS = (16384, 32768, 65536, 699051)

# one session family: share of single-turn sessions, turn counts, log-normal
# lengths of the first prompt and of each append (tokens), context cap
# (tokens), gap between turns (gamma shape, mean seconds), share of sessions
# that open with a shared system prompt; and about how many 16-token block
# accesses one session makes
FAMILIES = {
    "tiny": dict(single=0.30, turns=("geom", 0.2), first=(7.0, 1.0), append=(5.0, 1.0), cap=32768,
                 gap=(1.0, 30.0), sys=0.0, concurrency=12.0, per_session=1000),
    "chat": dict(single=0.40, turns=("zipf", 1.5, 200), first=(7.5, 1.2), append=(6.0, 1.0), cap=262144,
                 gap=(1.0, 30.0), sys=0.05, concurrency=256.0, per_session=11000),
    "agent": dict(single=0.0, turns=("pareto", 1.1, 2000), first=(7.0, 1.5), append=(7.0, 1.5), cap=131072,
                  gap=(4.0, 10.0), sys=0.0, concurrency=16.0, per_session=5500),
}


def listed():
    return [
        # one engine's few minutes of traffic, scored again and again while an
        # operator looks at it: tens of sessions, latency and launches count
        dict(name="tiny_access", kind="pipeline", family="tiny", accesses=64_773, block=16, residency="access",
             packed=False),
        # block keys of one scheduler step: 256 turns that extend known
        # prefixes (parent keys), the smallest call a server makes
        dict(name="turns_hash", kind="turns", requests=256, tokens=600, block=16),
        # a live window of keys reported by an engine, in a loop that may not allocate
        dict(name="window_noalloc", kind="window", accesses=1_000_003),
        # the agent trace at the serving block size and, for the granularity
        # sweep, at coarse blocks
        dict(name="agent_access", kind="pipeline", family="agent", accesses=27_647_805, block=16,
             residency="access", packed=False),
        dict(name="agent_b256_access", kind="pipeline", family="agent", accesses=1_719_571, block=256,
             residency="access", packed=False),
        # the chat trace
        dict(name="chat_access", kind="pipeline", family="chat", accesses=224_261_213, block=16, residency="access",
             packed=False),
        # chat and agent sessions mixed, the largest window that fits the card three times
        dict(name="mixed_access", kind="pipeline", family="mixed", accesses=800_000_017, block=16,
             residency="access", packed=False),
        # request-level residency over a log whose token streams are packed
        # without padding (starts at any token)
        dict(name="chat_request_packed", kind="pipeline", family="chat", accesses=60_000_001, block=16,
             residency="request", packed=True),
        # whole-session eviction
        dict(name="mixed_session", kind="pipeline", family="mixed", accesses=300_000_007, block=16,
             residency="session", packed=False),
        # workload characterisation
        dict(name="mixed_profile", kind="profile", family="mixed", accesses=200_000_003, block=16, packed=False),
        # block keys of any engine, no request table: generic stages
        dict(name="keys_generic", kind="keys", accesses=33_554_467),
        # the offline ceiling at every capacity
        dict(name="agent_belady", kind="belady", family="agent", accesses=4_000_037, block=16),
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["pipeline"] * 5 + ["profile", "keys", "window", "belady", "turns"])
    if kind == "turns":
        return dict(kind=kind, requests=log_int(1, 8192), tokens=log_int(32, 8192), block=rng.choice([16, 16, 32, 64, 24]))
    if kind == "window":
        return dict(kind=kind, accesses=log_int(1_000, 7_900_000))
    if kind == "keys":
        return dict(kind=kind, accesses=log_int(100_000, 150_000_000))
    if kind == "belady":
        return dict(kind=kind, family=rng.choice(["tiny", "agent", "chat"]), accesses=log_int(20_000, 4_000_000), block=16)
    family = rng.choice(["tiny", "chat", "agent", "mixed"])
    block = rng.choice([16, 16, 16, 32, 64, 128, 256, 24, 10])
    hi = 400_000_000 if block <= 32 else 400_000_000 * 16 // block
    case = dict(kind=kind, family=family, accesses=log_int(20_000, 2_000_000 if family == "tiny" else hi), block=block,
                packed=rng.random() < 0.3)
    if kind == "pipeline":
        case["residency"] = rng.choice(["access", "access", "request", "session"])
    return case


# ------------------------------------------------------------------ inputs

def _turn_counts(g, f, n):
    kind = f["turns"]
    if kind[0] == "geom":
        t = 1 + g.geometric(kind[1], size=n)
    elif kind[0] == "zipf":
        t = 1 + g.zipf(kind[1], size=n)
        while (bad := np.nonzero(t > kind[2])[0]).size:
            t[bad] = 1 + g.zipf(kind[1], size=bad.size)
    else:
        t = np.minimum(np.floor(1.0 + g.pareto(kind[1], size=n)), kind[2])
    return np.where(g.random(n) < f["single"], 1, t).astype(np.int64)


def _sessions(g, f, n):
    """Turns of n sessions of one family, session-major: session index, context
    tokens, seconds since the session's start; and which system prompt (-1: none)."""
    turns = _turn_counts(g, f, n)
    first_at = np.concatenate([[0], np.cumsum(turns)[:-1]])
    sess = np.repeat(np.arange(n), turns)
    m = sess.size
    is_first = np.zeros(m, bool)
    is_first[first_at] = True
    mu = np.where(is_first, f["first"][0], f["append"][0])
    sigma = np.where(is_first, f["first"][1], f["append"][1])
    add = np.maximum(1, np.rint(np.exp(mu + sigma * g.standard_normal(m)))).astype(np.int64)
    prompt = np.where(g.random(n) < f["sys"], g.integers(0, SYS_PROMPTS, size=n), -1)
    add[first_at] += np.where(prompt >= 0, SYS_LEN, 0)
    gap = np.where(is_first, 0.0, g.gamma(f["gap"][0], f["gap"][1] / f["gap"][0], size=m))
    ctx = np.cumsum(add)
    ctx -= np.repeat(ctx[first_at] - add[first_at], turns)
    at = np.cumsum(gap)
    at -= np.repeat(at[first_at], turns)
    keep = ctx <= f["cap"]               # contexts only grow: the session ends at its cap
    return sess[keep], ctx[keep], at[keep], prompt


def _log(case, seed):
    """The request table of a window of exactly ``accesses`` block accesses (host)."""
    g = np.random.Generator(np.random.PCG64(np.random.SeedSequence([seed, 11])))
    B, want = case["block"], case["accesses"]
    mix = [("chat", 0.7), ("agent", 0.3)] if case["family"] == "mixed" else [(case["family"], 1.0)]
    per = sum(w * FAMILIES[f]["per_session"] for f, w in mix) * 16 / B
    conc = max(FAMILIES[f]["concurrency"] for f, _ in mix)
    n = int(1.3 * want / per) + 8
    sess, ctx, ts, prompts, first = [], [], [], [], 0
    t_end, have = 0.0, 0
    while True:
        durations = []
        parts = []
        for f, w in mix:
            k = max(1, int(round(n * w)))
            s, c, a, p = _sessions(g, FAMILIES[f], k)
            last = np.zeros(k)
            np.maximum.at(last, s, a)
            durations.append(last)
            parts.append((s, c, a, p, k))
        rate = conc / max(1e-3, float(np.mean(np.concatenate(durations))))
        for s, c, a, p, k in parts:
            start = t_end + g.random(k) * (n / rate)      # Poisson starts, given their number
            sess.append(s + first)
            ctx.append(c)
            ts.append(start[s] + a)
            prompts.append(p)
            first += k
            have += int((c // B).sum())
        if have >= want:
            break
        t_end += n / rate
    sess, ctx, ts, prompts = (np.concatenate(x) for x in (sess, ctx, ts, prompts))
    order = np.lexsort((ctx, ts))
    sess, ctx, ts = sess[order], ctx[order], ts[order]
    cum = np.cumsum(ctx // B)
    r = int(np.searchsorted(cum, want, side="left")) + 1  # requests in the window
    sess, ctx, ts = sess[:r], ctx[:r].copy(), ts[:r]
    ctx[-1] -= (int(cum[r - 1]) - want) * B
    # one token stream per session, as long as its longest request here
    ids, sess = np.unique(sess, return_inverse=True)
    length = np.zeros(ids.size, np.int64)
    np.maximum.at(length, sess, ctx)
    room = length if case.get("packed") else (length + 3) // 4 * 4
    base = np.concatenate([[0], np.cumsum(room)]) + (1 if case.get("packed") else 0)
    off = np.concatenate([[0], np.cumsum(ctx // B)])
    assert off[-1] == want
    return dict(start=base[sess], length=ctx, off=off, session=sess, ts=np.rint(ts * 1e6).astype(np.int64),
                stream=base[:-1], stream_len=length, prompt=prompts[ids], tokens=int(base[-1]))


def _gen(seed, salt):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 1000003 + salt)
    return g


def _tokens(count, seed):
    return torch.randint(0, VOCAB, (count,), dtype=torch.int32, device="cuda", generator=_gen(seed, 1))


def _trace(case, seed):
    """The log on the GPU, as the entry points take it."""
    t = _log(case, seed)
    tokens = _tokens(t["tokens"], seed)
    prompts = torch.randint(0, VOCAB, (SYS_PROMPTS, SYS_LEN), dtype=torch.int32, device="cuda", generator=_gen(seed, 2))
    who = np.nonzero(t["prompt"] >= 0)[0]
    if who.size:
        col = torch.arange(SYS_LEN, device="cuda")
        start = torch.from_numpy(t["stream"][who]).cuda()
        have = torch.from_numpy(t["stream_len"][who]).cuda()
        src = prompts[torch.from_numpy(t["prompt"][who]).cuda()]
        ok = col[None, :] < have[:, None]
        tokens[(start[:, None] + col[None, :])[ok]] = src[ok]
    return dict(tokens=tokens, tok_start=torch.from_numpy(t["start"].astype(np.int64)).cuda(),
                tok_len=torch.from_numpy(t["length"].astype(np.int32)).cuda(),
                blk_off=torch.from_numpy(t["off"].astype(np.int64)).cuda(),
                session=torch.from_numpy(t["session"].astype(np.int32)).cuda(),
                ts_us=torch.from_numpy(t["ts"]).cuda())


def _mix64(z):
    """splitmix64's finalizer over int64 bit patterns (torch or numpy uint64)."""
    if isinstance(z, torch.Tensor):
        sr = lambda x, k: (x >> k) & ((1 << (64 - k)) - 1)                     # logical shift
        s64 = lambda v: v - (1 << 64) if v >= (1 << 63) else v
        z = (z ^ sr(z, 30)) * s64(0xBF58476D1CE4E5B9)
        z = (z ^ sr(z, 27)) * s64(0x94D049BB133111EB)
        return z ^ sr(z, 31)
    z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
    z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
    return z ^ (z >> np.uint64(31))


def _keys(case, seed):
    """A key stream: half of the accesses over a skewed popularity (rank
    log-uniform, so a few hot blocks), half over the whole population."""
    n = case["accesses"]
    distinct = max(2, n // 4)
    u = torch.rand(n, device="cuda", dtype=torch.float64, generator=_gen(seed, 3))
    rank = torch.exp(u * math.log(distinct)).to(torch.int64) - 1
    flat = torch.randint(0, distinct, (n,), device="cuda", generator=_gen(seed, 4))
    pick = torch.rand(n, device="cuda", generator=_gen(seed, 5)) < 0.5
    idx = torch.where(pick, rank.clamp_(0, distinct - 1), flat)
    return _mix64(idx * 7919 + (seed * 2654435761 + 12345))


def _turns(case, seed):
    g = np.random.Generator(np.random.PCG64(np.random.SeedSequence([seed, 12])))
    r, B = case["requests"], case["block"]
    # as many blocks whatever the seed: lengths vary around the mean and the
    # last turn takes what is left
    blocks = _turn_blocks(case)
    nb = np.maximum(0, np.rint(np.exp(g.normal(0.0, 0.7, size=r)) * blocks / r / 1.28)).astype(np.int64)
    off = np.minimum(np.concatenate([[0], np.cumsum(nb)]), blocks)
    off[-1] = blocks
    length = np.diff(off) * B + g.integers(0, B, size=r)
    start = np.concatenate([[0], np.cumsum((length + 3) // 4 * 4)])
    parent = g.integers(-2 ** 63, 2 ** 63 - 1, size=r, dtype=np.int64)
    return dict(tokens=_tokens(int(start[-1]) + 4, seed), tok_start=torch.from_numpy(start[:-1]).cuda(),
                tok_len=torch.from_numpy(length.astype(np.int32)).cuda(), blk_off=torch.from_numpy(off).cuda(),
                parent=torch.from_numpy(parent).cuda())


def _turn_blocks(case):
    return max(1, case["requests"] * case["tokens"] // case["block"])


def _caps(case):
    if case["kind"] in ("keys", "window"):
        lo, hi, extra = 2, 8, ()
    elif case["block"] != 16:             # granularity sweep: token capacities
        return np.array(sorted(int(round(10 ** (2 + 6 * k / 63))) // case["block"] for k in range(64)), np.uint64)
    else:
        lo, hi = (3, 7) if case["family"] == "chat" else (2, 8)
        extra = TABLE_BLOCKS
    pts = {int(round(10 ** (lo + (hi - lo) * k / 64))) for k in range(65)}
    return np.array(sorted(pts | set(extra)), np.uint64)


def _edges():
    """Reuse-interval and lifetime edges in microseconds: 1 ms to 10 days."""
    return np.array([int(round(10 ** (3 + 9 * k / 63))) for k in range(64)], np.uint64)


def _cost(case):
    B = case.get("block", 16)
    return ALPHA_PER_TOKEN * B, 2 * B * B


# ------------------------------------------------------------ the interface

def prepare(case, seed):
    kind = case["kind"]
    st = dict(kind=kind)
    if kind == "turns":
        st.update(_turns(case, seed), block=case["block"])
        n = _turn_blocks(case)
        st.update(n=n, keys=torch.empty(n, dtype=torch.int64, device="cuda"),
                  depth=torch.empty(n, dtype=torch.int32, device="cuda"),
                  ws=pc.workspace(pc.lib().pc_hash_blocks_ws(case["requests"])))
        return st
    if kind in ("keys", "window"):
        st["keys"] = _keys(case, seed)
        n = case["accesses"]
        st["caps"] = pc.to_dev_u64(_caps(case))
        k = st["caps"].numel()
        for name in ("prev", "next", "dist"):
            st[name] = torch.empty(n, dtype=torch.int32, device="cuda")
        st["bins"] = {b: torch.empty(k + 1, dtype=torch.int64, device="cuda")
                      for b in ("count", "depthsum", "cost_lo", "cost_hi", "nextuse")}
        st["ws_pn"] = pc.workspace(pc.lib().pc_prev_next_use_ws(n))
        if kind == "keys":
            st["ws_sd"] = pc.workspace(pc.lib().pc_stack_distance_ws(n))
        st["ws_mrc"] = pc.workspace(pc.lib().pc_mrc_weighted_ws(n, k))
        return st
    t = _trace(case, seed)
    n, B = case["accesses"], case["block"]
    caps = pc.to_dev_u64(_caps(case))
    alpha, beta = _cost(case)
    if kind == "profile":
        st["run"] = pc.Profiler(t["tokens"], t["tok_start"], t["tok_len"], t["blk_off"], n, t["session"], t["ts_us"],
                                pc.to_dev_u64(_edges()), block_size=B)
    else:
        st["run"] = pc.Pipeline(t["tokens"], t["tok_start"], t["tok_len"], t["blk_off"], n, caps, B, alpha, beta,
                                residency=case.get("residency", "access"), session=t["session"],
                                with_belady=kind == "belady")
    return st


def run(state):
    kind = state["kind"]
    if kind == "turns":
        keys, depth, _ = pc.hash_blocks(state["tokens"], state["tok_start"], state["tok_len"], state["blk_off"],
                                        state["n"], state["block"], parent=state["parent"], keys=state["keys"],
                                        depth=state["depth"], ws=state["ws"])
        return dict(keys=keys, depth=depth)
    if kind in ("keys", "window"):
        prev, nxt, dist = state["prev"], state["next"], state["dist"]
        pc.prev_next_use(state["keys"], prev, nxt, ws=state["ws_pn"])
        if kind == "keys":
            pc.stack_distance(prev, nxt, dist, ws=state["ws_sd"])
        else:
            pc.stack_distance_noalloc(prev, nxt, dist)
        pc.mrc_weighted(dist, state["caps"], nxt=nxt, out=state["bins"], ws=state["ws_mrc"])
        return dict(prev=prev, next=nxt, dist=dist, **state["bins"])
    p = state["run"]
    p.run()
    if kind == "profile":
        return dict(keys=p.keys, prev=p.prev, next=p.next, **p.reuse, **p.sessions)
    out = dict(keys=p.keys, prev=p.prev, dist=p.dist, **p.bins)
    if p.residency != "session":          # session-level eviction leaves next unspecified
        out["next"] = p.next
    if p.residency == "request":
        out["dist_req"] = p.dist_req
    if kind == "belady":
        out.update(min_hits=p.belady_out["hits"], min_depthsum=p.belady_out["depthsum"])
    return out


def work(case):
    """Bytes: the tokens of every request (each turn re-sends its context, and
    every re-sent context is input), the tables, and each result array; 8 for
    a key, 4 for a position, a distance or a depth.  Operations: nine 64-bit
    hash steps of ten integer operations per 16 tokens, a handful per access
    elsewhere, and one comparison per access and capacity for Belady's MIN."""
    kind = case["kind"]
    if kind == "turns":
        n = _turn_blocks(case)
        return dict(bytes=n * (4 * case["block"] + 12) + 28 * case["requests"], flops=n * (case["block"] // 2 + 1) * 10)
    n = case["accesses"]
    if kind in ("keys", "window"):
        return dict(bytes=n * (8 + 4 + 4 + 4), flops=n * 10)
    hashed = n * (4 * case["block"] + 8)
    ops = n * (case["block"] // 2 + 1) * 10
    if kind == "profile":
        return dict(bytes=hashed + 8 * n, flops=ops + 10 * n)
    per = {"access": 12, "request": 16, "session": 8}[case.get("residency", "access")]
    caps = _caps(case).size
    return dict(bytes=hashed + per * n + (4 * n if kind == "belady" else 0),
                flops=ops + 10 * n + (n * caps if kind == "belady" else 0))


def tolerance(case):
    return "exact"


# ---------------------------------------------------- the same from numpy

EXACT_MAX = 2_000_000


def exact(case, seed):
    """Keys, links, distances and bins in plain numpy, up to 2e6 accesses."""
    kind = case["kind"]
    if kind == "turns":
        n = _turn_blocks(case)
    else:
        n = case["accesses"]
    if n > EXACT_MAX or kind in ("profile", "belady") or case.get("residency", "access") != "access":
        return None
    if kind == "turns":
        t = {k: v.cpu().numpy() for k, v in _turns(case, seed).items()}
        keys, depth = _np_hash(t, case["block"], n, t["parent"].view(np.uint64))
        return dict(keys=keys.view(np.int64), depth=depth.astype(np.int32))
    if kind in ("keys", "window"):
        keys, depth, (alpha, beta) = _keys(case, seed).cpu().numpy().view(np.uint64), None, (1, 0)
    else:
        t = {k: v.cpu().numpy() for k, v in _trace(case, seed).items()}
        keys, depth = _np_hash(t, case["block"], n, None)
        alpha, beta = _cost(case)
    prev, nxt = _np_links(keys)
    dist = _np_distance(prev, nxt)
    out = dict(prev=prev, next=nxt, dist=dist)
    out = {k: np.where(v < 0, NONE, v).astype(np.uint32).view(np.int32) for k, v in out.items()}
    out.update(_np_bins(dist, nxt, depth, _caps(case).astype(np.int64), alpha, beta))
    if kind not in ("keys", "window"):
        out["keys"] = keys.view(np.int64)
    return out


def _np_hash(t, B, n, parent):
    """Chained keys, one block depth of every request at a time."""
    start, length, off = t["tok_start"], t["tok_len"].astype(np.int64), t["blk_off"]
    toks = t["tokens"].view(np.uint32).astype(np.uint64)
    step = lambda x, w: _mix64((x ^ w) + np.uint64(GOLDEN))
    nb = length // B
    keys, depth = np.zeros(n, np.uint64), np.zeros(n, np.int64)
    cur = np.zeros(nb.size, np.uint64) if parent is None else parent.copy()
    with np.errstate(over="ignore"):
        live = np.nonzero(nb > 0)[0]
        d = 0
        while live.size:
            h = np.zeros(live.size, np.uint64)
            for k in range(0, B, 2):
                at = start[live] + d * B + k
                h = step(h, toks[at] | toks[at + 1] << np.uint64(32))
            cur[live] = step(cur[live], h)
            keys[off[live] + d], depth[off[live] + d] = cur[live], d
            d += 1
            live = live[nb[live] > d]
    return keys, depth


def _np_links(keys):
    order = np.argsort(keys, kind="stable")
    same = keys[order][1:] == keys[order][:-1]
    prev, nxt = np.full(keys.size, -1, np.int64), np.full(keys.size, -1, np.int64)
    prev[order[1:][same]] = order[:-1][same]
    nxt[order[:-1][same]] = order[1:][same]
    return prev, nxt


def _np_distance(prev, nxt):
    """Earlier accesses whose block was last used before this one's, less the
    ones up to prev: a dominance count by merging blocks of doubling size."""
    n = prev.size
    v = prev + 1
    m = 1 << max(0, int(n - 1).bit_length())
    pos = np.argsort(np.concatenate([v, np.full(m - n, n + 1)]), kind="stable")   # positions in v order
    vs = np.concatenate([v, np.full(m - n, n + 1)])
    less = np.zeros(m, np.int64)
    lvl = 0
    while (1 << lvl) < m:
        # accesses grouped by block of 2^(lvl+1) positions, in v order inside it
        grp = pos >> (lvl + 1)
        o = pos[np.argsort(grp, kind="stable")]
        left = ((o >> lvl) & 1) == 0
        c = np.cumsum(left)
        g0 = (o >> (lvl + 1)) << (lvl + 1)
        base = np.where(g0 > 0, c[np.maximum(g0 - 1, 0)], 0)
        # lefts before this one in v order; cold ones (v = 0) come first, so they count as smaller
        right = ~left
        less[o[right]] += (c - base)[right]
        lvl += 1
    # for a warm access every cold one before it has a smaller v; warm v are distinct
    d = less[:n] - v
    return np.where(prev < 0, -1, d)


def _np_bins(dist, nxt, depth, caps, alpha, beta):
    k = caps.size
    t = np.arange(dist.size)
    bins = lambda x: np.where(x < 0, k, np.searchsorted(caps, np.maximum(x, 0), side="right"))
    b = bins(dist)
    count = np.bincount(b, minlength=k + 1)
    dsum = np.zeros(k + 1, np.int64)
    if depth is not None:
        np.add.at(dsum, b, depth)
    cost = [alpha * int(c) + beta * int(d) for c, d in zip(count, dsum)]
    as64 = lambda xs: np.array(xs, np.uint64).view(np.int64)
    return dict(count=count.astype(np.int64), depthsum=dsum, cost_lo=as64([c & (2 ** 64 - 1) for c in cost]),
                cost_hi=as64([c >> 64 for c in cost]),
                nextuse=np.bincount(bins(np.where(nxt < 0, -1, nxt - t)), minlength=k + 1).astype(np.int64))
