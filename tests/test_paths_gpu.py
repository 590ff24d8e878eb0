"""The size rules inside prev / next and the stack distance, at the sizes where
they change: the sort's tiles, run counts around a merge block of 2048 and its eightfolds, the
dominance count as one launch and as several, the passes over the high key
bits, and the generic prev / next behind the chained one as one launch and as
several; and the bins where their value classes, chunks and workgroup sizes
change.  All results are whole numbers and must match exactly."""
import numpy as np
import pytest
import torch

import oracle
from paper_2609_28870_amd import pc

pytestmark = pytest.mark.gpu
MIX = 0x9E3779B97F4A7C15


def device_keys(n, kinds, low_shared=False, seed=3):
    """n keys drawn from `kinds` values; low_shared: all of them agree in most
    of their low bits, so the sort has to look at the high ones."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    idx = torch.randint(0, kinds, (n,), device="cuda", generator=g)
    return (idx << 32) | (idx % 5) if low_shared else idx * (MIX - (1 << 64)) ^ (idx << 17)


@pytest.mark.parametrize("runs", [1, 255, 2047, 2048, 2049, 4097, 16383, 16384, 16385, 131073])
def test_run_counts_around_the_merge_blocks(runs):
    # 8 * runs fresh keys, then the same keys again in pieces of 8, whose order
    # is shuffled with no two pieces left in sequence: exactly `runs` runs
    rng = np.random.default_rng(runs)
    order = rng.permutation(runs)
    for _ in range(64):
        bad = np.nonzero(np.diff(order) == 1)[0]
        if bad.size == 0:
            break
        other = rng.integers(0, runs, bad.size)
        for b, o in zip(bad, other):
            order[b], order[o] = order[o], order[b]
    again = (order[:, None] * 8 + np.arange(8)).reshape(-1)
    keys = np.concatenate([np.arange(8 * runs), again]).astype(np.uint64)
    p, q = oracle.prev_next(keys)
    pd = torch.from_numpy(p.view(np.int32)).cuda()
    nd = torch.from_numpy(q.view(np.int32)).cuda()
    dd, ws = pc.stack_distance_runs(pd, nd)
    info = pc.runs_info(ws)
    assert info["runs"] == int((np.diff(order) != 1).sum()) + 1 and not info["generic"], info
    assert pc.workspace_status(ws) == 0
    assert np.array_equal(pc.as_u32(dd), oracle.stack_distance_bit(p))


@pytest.mark.parametrize("n", [257, 65_537, (1 << 20) + 1, (1 << 22) - 1, 1 << 22, (1 << 22) + 1])
def test_the_dominance_count_behind_the_runs(n):
    # random keys have too many runs; past the window of the first level too
    prev, nxt, _ = pc.prev_next_use(device_keys(n, max(2, n // 4)))
    dist, ws = pc.stack_distance_runs(prev, nxt)
    assert pc.runs_info(ws)["generic"] == (n > 2048) and pc.workspace_status(ws) == 0
    want = oracle.stack_distance_bit(pc.as_u32(prev))
    assert np.array_equal(pc.as_u32(dist), want)
    plain = pc.stack_distance(prev, nxt)
    plain = plain[0] if isinstance(plain, tuple) else plain
    assert np.array_equal(pc.as_u32(plain), want)


@pytest.mark.parametrize("n", [1500, 8191, 8192, 8193, 100_003, (1 << 20) + 3])
def test_high_key_bits(n):
    keys = device_keys(n, max(2, n // 4), low_shared=True)
    prev, nxt, ws = pc.prev_next_use(keys)
    p, q = oracle.prev_next(keys.cpu().numpy().view(np.uint64))
    assert pc.high_key_passes_ran(ws) and pc.workspace_status(ws) == 0
    assert np.array_equal(pc.as_u32(prev), p) and np.array_equal(pc.as_u32(nxt), q)


@pytest.mark.parametrize("n", [1, 2047, 2048, 2049, 4097, (1 << 18) - 1, 1 << 18, (1 << 18) + 1, (1 << 20) - 1, 1 << 20,
                               (1 << 20) + 1, (1 << 20) + 8193])
def test_sort_tile_sizes(n):
    keys = device_keys(n, max(2, n // 3))
    prev, nxt, ws = pc.prev_next_use(keys)
    p, q = oracle.prev_next(keys.cpu().numpy().view(np.uint64))
    assert pc.workspace_status(ws) == 0
    assert np.array_equal(pc.as_u32(prev), p) and np.array_equal(pc.as_u32(nxt), q)


@pytest.mark.parametrize("n", [(1 << 22) + 1, (1 << 22) + 57_344, (1 << 22) + 65_535, (1 << 22) + 65_536,
                               (1 << 22) + 65_537])
def test_tiles_of_a_later_partition_pass(n):
    """Above 2^22 keys the way back to time order has a later pass, whose
    8192-element tiles are dealt in eighths: 513, 519, 520 and 521 tiles."""
    keys = device_keys(n, n // 3)
    prev, nxt, ws = pc.prev_next_use(keys)
    p, q = oracle.prev_next(keys.cpu().numpy().view(np.uint64))
    assert pc.workspace_status(ws) == 0
    assert np.array_equal(pc.as_u32(prev), p) and np.array_equal(pc.as_u32(nxt), q)


def test_a_larger_call_never_needs_less_workspace():
    sizes = [pc.lib().pc_prev_next_use_ws(n) for k in (11, 18, 20, 21, 22) for n in range((1 << k) - 8200, (1 << k) + 8200, 511)
             if n > 0]
    assert sizes == sorted(sizes)


@pytest.mark.parametrize("n,low_shared",
                         [(n, False) for n in (1, 777, 8193, (1 << 20) - 1, 1 << 20, (1 << 24) + 1, (1 << 26) - 1,
                                               1 << 26)] +
                         [(n, True) for n in (777, 8193, (1 << 20) - 1, 1 << 20)])
def test_the_generic_path_behind_the_chained_one(n, low_shared):
    keys = device_keys(n, max(2, n // 4), low_shared)
    reqs = max(1, n // 50)
    off = torch.arange(reqs + 1, device="cuda") * n // reqs
    prev, nxt, ws = pc.prev_next_chained(keys, off)
    info = pc.chained_info(ws)
    assert pc.workspace_status(ws) == 0
    if n > 8:
        assert info["generic"], info
    want_prev, want_next, _ = pc.prev_next_use(keys)
    assert torch.equal(prev, want_prev) and torch.equal(nxt, want_next)
    if n <= 1 << 20:
        p, q = oracle.prev_next(keys.cpu().numpy().view(np.uint64))
        assert np.array_equal(pc.as_u32(prev), p) and np.array_equal(pc.as_u32(nxt), q)


@pytest.mark.parametrize("n", [2047, 2049, 3000, 20_000, 65_535, 65_537, 262_145])
@pytest.mark.parametrize("low_shared", [False, True])
def test_one_launch_paths_with_more_workgroups_than_tiles(n, low_shared):
    # up to 32 workgroups where the sort and the dominance count have a few
    # tiles: some get none of a phase's chunks
    keys = device_keys(n, max(2, n // 4), low_shared)
    reqs = n // 50
    off = torch.arange(reqs + 1, device="cuda") * n // reqs
    prev, nxt, ws = pc.prev_next_chained(keys, off)
    p, q = oracle.prev_next(keys.cpu().numpy().view(np.uint64))
    assert pc.chained_info(ws)["generic"] and pc.workspace_status(ws) == 0
    assert np.array_equal(pc.as_u32(prev), p) and np.array_equal(pc.as_u32(nxt), q)
    dist, ws = pc.stack_distance_runs(prev, nxt)
    assert pc.workspace_status(ws) == 0
    assert np.array_equal(pc.as_u32(dist), oracle.stack_distance_bit(p))


@pytest.mark.parametrize("edges", ["classes", "one octave", "one edge", "top"])
@pytest.mark.parametrize("n,shift", [(1, 0), (15, 1), (1 << 16, 3), ((1 << 20) + 1, 0), ((1 << 20) + 7, 2), (4_300_003, 1),
                                     (9_000_001, 0)])
def test_bins_of_values_around_the_edges(n, shift, edges):
    # distances and next-use gaps on both sides of class starts (32 classes to
    # an octave) and of edges, NONE among them; views at any 4-byte alignment
    rng = np.random.default_rng(n)
    starts = np.array([0, 1, 31, 32, 33] + [(32 + k) << e for e in range(1, 27) for k in (0, 1, 31)], np.uint64)
    caps = {"classes": starts,
            "one octave": np.sort(rng.integers(1 << 15, 1 << 16, 900)).astype(np.uint64),
            "one edge": np.array([1 << 15], np.uint64),
            "top": np.array([0, 2 ** 32 - 2, 2 ** 32 - 1, 2 ** 32, 2 ** 40], np.uint64)}[edges]
    near = (np.concatenate([starts, caps, [2 ** 32 - 2, 2 ** 32]])[:, None] + np.array([-1, 0, 1], np.int64)).reshape(-1)
    near = np.clip(near.astype(np.int64), 0, 2 ** 32 - 1)
    d = near[rng.integers(0, near.size, n)]
    dep = rng.integers(0, 1 << 20, n)
    t = np.arange(n, dtype=np.int64)
    gap = near[rng.integers(0, near.size, n)]
    nxt = np.where((gap > 0) & (t + gap < 2 ** 32 - 1), t + gap, 2 ** 32 - 1)      # NONE: no next use
    gap = np.where(nxt == 2 ** 32 - 1, 2 ** 32 - 1, nxt - t)
    view = lambda a: pc.to_dev_u32(np.concatenate([np.zeros(shift), a]).astype(np.uint32))[shift:]
    out, ws = pc.mrc_weighted(view(d), pc.to_dev_u64(caps), view(dep), view(nxt), 3, 2)
    assert pc.workspace_status(ws) == 0
    got = pc.bins_to_host(out)

    def hist(x, w=None):   # NONE lies past every edge
        b = np.where(x == 2 ** 32 - 1, caps.size, np.searchsorted(caps.astype(np.int64), x, side="right"))
        full = np.zeros(caps.size + 1, object)
        for k in np.unique(b):
            full[k] = int((b == k).sum()) if w is None else int(w[b == k].sum())
        return full.tolist()

    count, depthsum = hist(d), hist(d, dep)
    assert [int(x) for x in got["count"]] == count and [int(x) for x in got["depthsum"]] == depthsum
    assert [int(x) for x in got["cost"]] == [3 * a + 2 * b for a, b in zip(count, depthsum)]
    assert [int(x) for x in got["nextuse"]] == hist(gap)


def periodic(n, period, key_of, step=1 << 26):
    """keys[t] = key_of(t mod period), and a check of prev / next against t - period / t + period."""
    keys = torch.empty(n, dtype=torch.int64, device="cuda")
    for a in range(0, n, step):
        keys[a:a + step] = key_of(torch.arange(a, min(a + step, n), device="cuda") % period)

    def check(prev, nxt):
        for a in range(0, n, step):
            t = torch.arange(a, min(a + step, n), device="cuda")
            back, ahead = t - period, t + period
            back[back < 0] = pc.NONE
            ahead[ahead >= n] = pc.NONE
            assert torch.equal(prev[a:a + step].to(torch.int64) & 0xFFFFFFFF, back), a
            assert torch.equal(nxt[a:a + step].to(torch.int64) & 0xFFFFFFFF, ahead), a
    return keys, check


@pytest.mark.parametrize("n", [1 << 26, (1 << 26) + 8193])
def test_high_key_bits_inside_the_one_launch_path(n):
    # from 2^26 keys on the generic path behind the chained one is one launch
    # again, here with its passes over the high key bits
    keys, check = periodic(n, (1 << 24) + 5, lambda i: (i << 32) | (i % 4099))
    reqs = n // 70
    off = torch.arange(reqs + 1, device="cuda") * n // reqs
    prev, nxt, ws = pc.prev_next_chained(keys, off)
    info = pc.chained_info(ws)
    assert pc.workspace_status(ws) == 0 and info["generic"] and info["high_anchor"], info
    check(prev, nxt)


def test_persistent_launches_on_two_streams_at_once():
    # their phases wait for chunks, which only running workgroups hold
    n, sides = 300_007, []
    off = torch.arange(n // 50 + 1, device="cuda") * n // (n // 50)
    for seed in (1, 2):
        keys = device_keys(n, n // 4, low_shared=seed == 2, seed=seed)
        p, q = oracle.prev_next(keys.cpu().numpy().view(np.uint64))
        outs = [torch.empty(n, dtype=torch.int32, device="cuda") for _ in range(3)]
        sides.append((keys, p, q, oracle.stack_distance_bit(p), outs,
                      pc.workspace(pc.lib().pc_prev_next_chained_ws(n, off.numel() - 1)),
                      pc.workspace(pc.lib().pc_stack_distance_runs_ws(n)), torch.cuda.Stream()))
    torch.cuda.synchronize()
    for _ in range(5):
        for keys, _, _, _, (prev, nxt, dist), ws_pn, ws_sd, stream in sides:
            with torch.cuda.stream(stream):
                pc.prev_next_chained(keys, off, prev, nxt, ws_pn)
                pc.stack_distance_runs(prev, nxt, dist, ws_sd)
    torch.cuda.synchronize()
    for _, p, q, d, (prev, nxt, dist), ws_pn, ws_sd, _ in sides:
        assert pc.workspace_status(ws_pn) == 0 and pc.workspace_status(ws_sd) == 0
        assert pc.chained_info(ws_pn)["generic"] and pc.runs_info(ws_sd)["generic"]
        assert np.array_equal(pc.as_u32(prev), p) and np.array_equal(pc.as_u32(nxt), q)
        assert np.array_equal(pc.as_u32(dist), d)


def test_prev_next_above_2e31_keys():
    # 18 bits above the last step's ranges: a link and two later partition passes
    n = (1 << 31) + 12_345
    keys, check = periodic(n, 700_000_001, lambda i: i * (MIX - (1 << 64)))
    prev, nxt, ws = pc.prev_next_use(keys)
    assert pc.workspace_status(ws) == 0 and not pc.high_key_passes_ran(ws)
    del keys
    check(prev, nxt)
