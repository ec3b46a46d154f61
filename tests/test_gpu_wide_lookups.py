"""Lookups of few contexts whose 257 .. 1024 survivors are followed up to sixteen to a lane, and the counts beyond, which are streamed, against
the oracle, exactly: texts that agree for a while, that all differ, pool and own text mixed."""
import numpy as np
import pytest

from tests.test_gpu_lane_votes import _flat_pool, _pool
from tests.test_gpu_retrieval import _compare as compare_pool
from tests.test_gpu_temp_branch import _compare as compare_own

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("count", [257, 700, 1023, 1024, 1025, 1500])
@pytest.mark.parametrize("vocab", [2, 1000])
@pytest.mark.parametrize("K", [1, 2, 4, 9, 33])
def test_counts_up_to_sixteen_waves(count, vocab, K):
    rng = np.random.default_rng(count * 100 + K + vocab)
    toks, off, keys, _ = _pool(rng, count, vocab)
    compare_pool(toks, off, keys, [3, 3, 4], [[1, 7], [toks[0], toks[1]], [1, 7]], 1, 2, K)


@pytest.mark.parametrize("count", [900, 1024])
@pytest.mark.parametrize("agree", [0, 3, 9])
@pytest.mark.parametrize("spread", [5, 100, 5000])
def test_votes_over_many_tokens(count, agree, spread):
    rng = np.random.default_rng(count + 10 * agree + spread)
    pool = _flat_pool(rng, count, agree, spread)
    compare_pool(pool[0], pool[1], pool[2], [3, 3], [[1, 7], [1, 7]], 1, 2, 16)


def _tokens_of_hashes(first, count):
    """The tokens (>= 0) whose hash in the vote table is one of `count` neighbouring values: the mixer's inverse."""
    h = np.arange(first, first + count, dtype=np.uint64)
    mask = np.uint64(0xFFFFFFFF)
    for shift, factor in ((16, 0xC2B2AE35), (13, 0x85EBCA6B), (16, None)):
        x = h
        for _ in range(32 // shift):
            x = h ^ (x >> np.uint64(shift))
        h = x if factor is None else (x * np.uint64(pow(factor, -1, 1 << 32))) & mask
    return h[h < 1 << 31].astype(np.int64)


def test_tokens_of_hashes():
    t = _tokens_of_hashes(5 << 10, 1024).astype(np.uint64)
    mask = np.uint64(0xFFFFFFFF)
    h = t ^ (t >> np.uint64(16))
    h = (h * np.uint64(0x85EBCA6B)) & mask
    h ^= h >> np.uint64(13)
    h = (h * np.uint64(0xC2B2AE35)) & mask
    h ^= h >> np.uint64(16)
    assert len(t) > 400 and (h >> np.uint64(10) == 5).all()


@pytest.mark.parametrize("form", ["pool", "own"])
@pytest.mark.parametrize("count", [900, 1024, 1025, 1600])
def test_votes_over_tokens_that_share_their_upper_hash_bits(count, form):
    """More different successors than the table may hold, all with the same upper bits: parts of the vote by those bits alone would never
    be small enough."""
    rng = np.random.default_rng(count)
    tokens = _tokens_of_hashes(5 << 10, 1024)
    pick = np.concatenate([tokens, rng.choice(tokens, count - len(tokens))])
    toks = np.stack([np.full(count, 7), pick, pick[::-1]], 1).reshape(-1).astype(np.int32)
    off, keys = np.arange(count + 1, dtype=np.int64) * 3, np.full(count, 3, dtype=np.int64)
    if form == "pool":
        compare_pool(toks, off, keys, [3, 3], [[1, 7], [1, 7]], 1, 2, 3)
    else:
        own = np.stack([np.full(300, 7), rng.choice(tokens, 300)], 1).reshape(-1).tolist() + [5, 7]
        compare_own(toks, off, keys, [3, 3], [own, [5, 7]], 1, 2, 3)


@pytest.mark.parametrize("count", [400, 1000, 1020, 1024])
def test_pool_and_own_text_beyond_four_waves(count):
    rng = np.random.default_rng(count)
    toks, off, keys, trunk = _pool(rng, count, 2)
    owns = []
    for reps in (0, 3, 5, 24, 70):
        own = []
        for _ in range(reps):
            own += [7] + trunk[:int(rng.integers(1, 12))].tolist()
        owns.append(own + [5, 7])
    compare_own(toks, off, keys, [3, 3, 3, 3, 9], owns, 1, 2, 12)


def test_runs_that_split_at_once_take_no_longer_than_shorter_ones():
    """512 occurrences whose first vote leaves about 25 against 200 that lanes follow throughout: followed sixteen to a lane they took
    2.4 times as long, behind a vote by the table three quarters as long."""
    import time

    import torch

    import paper_2408_05676_amd as laser
    rng = np.random.default_rng(0)
    trunk, K, B, took = rng.integers(100, 30000, 40), 16, 256, []
    for count in (200, 512):
        seqs = [np.concatenate([[7], np.roll(trunk, i % 20)[:int(rng.integers(20, 41))]]) for i in range(count)]
        off = np.cumsum([0] + [len(s) for s in seqs]).astype(np.int64)
        pool = laser.Pool(np.concatenate(seqs).astype(np.int32), off, np.full(count, 3, np.int64), 2)
        keys = torch.full((B,), 3, dtype=torch.int64, device="cuda")
        tail = torch.tensor([[1, 7]] * B, dtype=torch.int32, device="cuda")
        best = 1e9
        for _ in range(5):
            torch.cuda.synchronize()
            t = time.perf_counter()
            for _ in range(100):
                laser.retrieve_drafts(pool, keys, tail, 1, 2, K, 1)
            torch.cuda.synchronize()
            best = min(best, (time.perf_counter() - t) / 100)
        took.append(best)
        pool.close()
    assert took[1] <= 1.5 * took[0], took
