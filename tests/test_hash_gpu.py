"""pc_hash_blocks where its pipeline of rounds can go wrong: requests around
the round lengths (64, 128 and 256 blocks), empty ones among them, request
counts on either side of the rows a workgroup holds (later requests come from
the counter), block sizes with a short last chunk of tokens, streams that
start at any token, both block orders, parents, depths and the histogram."""
import numpy as np
import pytest
import torch

import oracle
from paper_2609_28870_amd import pc

pytestmark = pytest.mark.gpu


def check(blocks, B, seed, deepest=False, parent=False, pad=0, ws=None):
    g = np.random.default_rng(seed)
    blocks = np.asarray(blocks, np.int64)
    length = blocks * B + g.integers(0, B, size=blocks.size)
    start = pad + np.concatenate([[0], np.cumsum(length)[:-1]])      # packed: any 4-byte alignment
    tokens = g.integers(0, 151936, size=int(start[-1] + length[-1]), dtype=np.int32)   # ends with the last request
    par = g.integers(0, 2 ** 63, size=blocks.size).astype(np.uint64) if parent else None
    want, depth = oracle.hash_requests(tokens, start, length, B, parent=par, root=5)
    off = np.concatenate([[0], np.cumsum(blocks)]).astype(np.uint64)
    if deepest:
        at = np.repeat(off[:-1] + off[1:] - np.uint64(1), blocks) - np.arange(off[-1], dtype=np.uint64)
        want, depth = want[at.astype(np.int64)], depth[at.astype(np.int64)]
    hist = torch.full((1024,), -1, dtype=torch.int32, device="cuda")
    keys, dep, ws = pc.hash_blocks(torch.from_numpy(tokens).cuda(), pc.to_dev_u64(start), pc.to_dev_u32(length),
                                   pc.to_dev_u64(off), int(off[-1]), B,
                                   parent=None if par is None else pc.to_dev_u64(par), root=5, key_hist=hist,
                                   deepest_first=deepest, ws=ws)
    assert pc.workspace_status(ws) == 0
    assert np.array_equal(pc.as_u64(keys), want)
    assert np.array_equal(pc.as_u32(dep), depth)
    low = np.concatenate([np.bincount(((want >> np.uint64(8 * p)) & np.uint64(255)).astype(np.int64), minlength=256)
                          for p in range(4)])
    assert np.array_equal(pc.as_u32(hist).astype(np.int64), low)


EDGES = [0, 1, 2, 15, 16, 17, 63, 64, 65, 0, 127, 128, 129, 191, 255, 256, 257, 320, 511, 512, 513, 1, 0]


@pytest.mark.parametrize("B", [2, 10, 16, 24, 32, 48, 80, 144, 256, 1024])
def test_block_counts_around_the_round_lengths(B):
    check(EDGES, B, B, deepest=B % 32 == 0, parent=B % 48 == 0, pad=B % 3)


@pytest.mark.parametrize("n_seqs,B", [(1, 16), (513, 16), (4096, 16), (4097, 16), (20000, 16), (32769, 16), (70001, 16),
                                      (70001, 2), (9000, 64), (5000, 256)])
def test_request_counts_around_the_rows_in_flight(n_seqs, B):
    g = np.random.default_rng(n_seqs)
    blocks = np.minimum(g.geometric(0.15, size=n_seqs) - 1, 90)      # a fair share of empty requests
    blocks[g.integers(0, n_seqs, size=3)] = [300, 700, 65]
    check(blocks, B, n_seqs, deepest=n_seqs % 2 == 1, parent=n_seqs % 3 == 0, pad=1)


@pytest.mark.parametrize("n_seqs,mean,B", [(9000, 520, 16), (13000, 400, 16), (17000, 300, 16), (40000, 120, 16),
                                           (70001, 70, 16), (40000, 70, 24), (5000, 110, 128), (33000, 17, 128),
                                           (17000, 17, 256), (4097, 9, 256), (8200, 36, 256)])
def test_requests_ordered_by_length(n_seqs, mean, B):
    # enough tokens for the order, at request counts on both sides of each rule
    # on the rows in flight; lengths spread over many length classes
    g = np.random.default_rng(n_seqs + B)
    blocks = np.minimum(g.geometric(1 / mean, size=n_seqs), 40 * mean)
    blocks[g.integers(0, n_seqs, size=3)] = [0, 1, 31]
    check(blocks, B, n_seqs, deepest=n_seqs % 2 == 1, parent=n_seqs % 5 != 0, pad=1)
    if n_seqs == 9000:      # a workspace without room for the order is enough
        check(blocks, B, n_seqs, ws=pc.workspace(512))


def test_a_bad_request_is_skipped_and_reported():
    tokens = torch.arange(4096, dtype=torch.int32, device="cuda")
    keys = torch.full((200,), 7, dtype=torch.int64, device="cuda")
    start, length, off = np.array([0, 4000, 64]), np.array([64, 128, 3200]), np.array([0, 4, 12, 212])
    _, _, ws = pc.hash_blocks(tokens, pc.to_dev_u64(start), pc.to_dev_u32(length), pc.to_dev_u64(off), 200, 16,
                              want_depth=False, keys=keys)
    assert pc.workspace_status(ws) == 2      # one past the tokens, one past the blocks
    want, _ = oracle.hash_requests(np.arange(4096, dtype=np.int32), start[:1], length[:1], 16)
    assert np.array_equal(pc.as_u64(keys)[:4], want) and (pc.as_u64(keys)[4:] == 7).all()


@pytest.mark.parametrize("n_seqs,B,most", [(1 << 19, 16, 9), (1 << 19, 16, 60), ((1 << 19) - 1, 16, 9), (1 << 19, 24, 9),
                                           (1 << 19, 24, 40), (1 << 16, 10, 200), (1 << 13, 32, 60), ((1 << 13) - 1, 32, 40),
                                           (1 << 11, 64, 40), ((1 << 11) - 1, 64, 40), (1 << 16, 64, 60),
                                           (1 << 16, 128, 20), (1 << 13, 128, 40), (1 << 15, 256, 26), (1 << 15, 256, 52)])
def test_short_requests_share_the_sweeps(n_seqs, B, most):
    # on both sides of each rule on the number and the mean length of short
    # requests; a few long ones among them leave most sweeps of a round empty
    g = np.random.default_rng(n_seqs + B + most)
    blocks = g.integers(0, most + 1, size=n_seqs)
    blocks[g.integers(0, n_seqs, size=4)] = [700, 257, 64, 65]
    check(blocks, B, most, deepest=B % 3 == 0, parent=B != 24, pad=1)
