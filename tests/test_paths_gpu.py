"""The size rules inside prev / next and the stack distance, at the sizes where
they change: run counts around a merge block of 2048 and its eightfolds, the
dominance count as one launch and as several, the passes over the high key
bits, and the generic prev / next behind the chained one as one launch and as
several.  All results are whole numbers and must match exactly."""
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
