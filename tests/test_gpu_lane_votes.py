"""Lookups whose survivors are followed by a wavefront's lanes, against the oracle, exactly: suffixes with just under, at and over 64,
256 and 512 occurrences, pool and own text mixed, chains shorter and longer than the tokens requested at a time."""
import numpy as np
import pytest

from tests.test_gpu_retrieval import _compare as compare_pool
from tests.test_gpu_temp_branch import _compare as compare_own
from tests.test_gpu_tree import _check_trees as compare_trees

pytestmark = pytest.mark.gpu


def _pool(rng, count, vocab):
    """`count` occurrences of the token 7 followed by texts of 0..40 tokens that agree for a while; some end at once."""
    trunk = rng.integers(8, 8 + vocab, 40)
    seqs = []
    for _ in range(count):
        t = trunk.copy()
        cut = int(rng.integers(0, 41))
        t[cut:] = rng.integers(8, 8 + vocab, 40 - cut)
        seqs.append([7] + t[:max(1, int(rng.integers(0, 41)))].tolist())
    off = np.cumsum([0] + [len(s) for s in seqs]).astype(np.int64)
    return np.concatenate(seqs).astype(np.int32), off, np.full(count, 3, np.int64), trunk


@pytest.mark.parametrize("count", [1, 2, 63, 64, 65, 255, 256, 257, 512, 513])
@pytest.mark.parametrize("K", [1, 8, 9, 16, 63])
def test_counts_around_a_wave(count, K):
    rng = np.random.default_rng(count * 100 + K)
    toks, off, keys, _ = _pool(rng, count, 3)
    compare_pool(toks, off, keys, [3, 3, 4], [[1, 7], [toks[0], toks[1]], [1, 7]], 1, 2, K)
    compare_pool(toks, off, keys, [3], [[1, 7]], 1, 2, K, mt=min(K, 5))


@pytest.mark.parametrize("count", [1, 40, 62, 63, 64, 200, 254, 255])
@pytest.mark.parametrize("vocab", [2, 1000])
def test_pool_and_own_text_share_the_lanes(count, vocab):
    rng = np.random.default_rng(count + vocab)
    toks, off, keys, trunk = _pool(rng, count, vocab)
    owns = []
    for reps in (0, 1, 2, 24, 70):
        own = []
        for _ in range(reps):
            own += [7] + trunk[:int(rng.integers(1, 12))].tolist()
        owns.append(own + [5, 7])
    compare_own(toks, off, keys, [3, 3, 3, 3, 9], owns, 1, 2, 12)


@pytest.mark.parametrize("count", [1, 63, 64, 65, 255, 256, 257])
@pytest.mark.parametrize("K", [1, 8, 32])
@pytest.mark.parametrize("vocab", [2, 1000])
def test_trees_around_four_waves(count, K, vocab):
    rng = np.random.default_rng(count * 100 + K + vocab)
    toks, off, keys, _ = _pool(rng, count, vocab)
    compare_trees((toks, off, keys), [[1, 7], toks[:2].tolist(), [5]], [3, 3, 3], 1, 2, K)
    compare_trees((toks, off, keys), [[1, 7]], [3], 1, 2, K, min_tokens=min(K, 5))


def _flat_pool(rng, count, agree, spread):
    """`count` texts after the token 7 that agree for `agree` tokens, then fan out over about `spread` tokens, then agree again."""
    trunk = rng.integers(8, 40, 12)
    seqs = []
    for i in range(count):
        t = trunk.tolist()
        t[agree] = 100 + int(rng.integers(0, spread)) if spread < count else 100 + i
        seqs.append([7] + t[:12 - i % 3])
    return np.concatenate(seqs).astype(np.int32), np.cumsum([0] + [len(s) for s in seqs]).astype(np.int64), np.full(count, 3, np.int64), trunk


@pytest.mark.parametrize("count", [64, 65, 200, 256, 257])
@pytest.mark.parametrize("agree,spread", [(0, 8), (0, 9), (0, 10), (0, 1000), (1, 60), (2, 1000), (7, 40), (8, 1000), (9, 9)])
def test_votes_over_many_tokens(count, agree, spread):
    """Votes that stay open after eight ballots, at the first step, inside, at the end and behind the tokens requested at a time."""
    rng = np.random.default_rng(count * 10 + agree + spread)
    toks, off, keys, trunk = _flat_pool(rng, count, agree, spread)
    for K in (1, 2, 4, 5, 9, 11):
        compare_pool(toks, off, keys, [3, 3], [[1, 7], [7, trunk[0]]], 1, 2, K)
    own = [7] + trunk[:6].tolist() + [7] + trunk[:agree].tolist() + [101, 5, 7]
    compare_own(toks, off, keys, [3, 3, 3], [own, own[8:], [7]], 1, 2, 10)


def test_a_vote_over_many_tokens_takes_no_longer_in_the_lanes():
    """256 occurrences with successors of their own (the lanes) against 257 (the vote table): ballots alone took three times as long."""
    import time

    import torch

    import paper_2408_05676_amd as laser
    took = []
    for count in (256, 257):
        toks, off, keys, _ = _flat_pool(np.random.default_rng(1), count, 0, 1000)
        pool = laser.Pool(toks, off, keys, 2)
        B, K = 2048, 2
        i32 = dict(dtype=torch.int32, device="cuda")
        args = (pool, torch.full((B,), 3, dtype=torch.int64, device="cuda"), torch.tensor([[1, 7]] * B, **i32), 1, 2, K, 1)
        out = (torch.empty((B, K), **i32), torch.empty(B, **i32), torch.empty(B, **i32), torch.empty(B, dtype=torch.int64, device="cuda"))
        best = 1e9
        for _ in range(6):
            torch.cuda.synchronize()
            t = time.perf_counter()
            for _ in range(40):
                laser.retrieve_drafts(*args, out=out)
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t)
        took.append(best)
        pool.close()
    assert took[0] <= 1.6 * took[1], took


def test_long_runs_of_more_than_1024_contexts():
    """Beyond 1024 contexts a streamed run is voted on in groups of 64: the same results as for few contexts, chains and own text."""
    import torch

    import paper_2408_05676_amd as laser
    rng = np.random.default_rng(4)
    count, K = 700, 12
    toks, off, keys, trunk = _pool(rng, count, 3)
    pool = laser.Pool(toks, off, keys, 2)
    tails = np.array([[1, 7], [7, trunk[0]], [1, 5], [7, int(toks[1])]], np.int32)
    own = np.full((4, 64), 7, np.int32)
    own[:, 1::2] = rng.integers(8, 12, (4, 32))
    got = []
    for reps in (1, 257):                                       # 4 and 1028 contexts
        dev = lambda a: torch.tensor(np.tile(a, (reps,) + (1,) * (a.ndim - 1)), device="cuda")
        qk, tail = dev(np.full(4, 3, np.int64)), dev(tails)
        got.append([[t.cpu().numpy() for t in laser.retrieve_drafts(pool, qk, tail, 1, 2, K, 1)],
                    [t.cpu().numpy() for t in laser.retrieve_drafts_temp(pool, qk, tail, dev(own), dev(np.full(4, 64, np.int32)), 1, 2, K, 1)]])
    for few, many in zip(*got):
        for x, y in zip(few, many):
            assert (np.tile(x, (257,) + (1,) * (x.ndim - 1)) == y).all()
    compare_pool(toks, off, keys, [3] * 4, tails.tolist(), 1, 2, K)
    pool.close()


def test_many_contexts_over_a_long_run_take_no_longer_together():
    """2048 contexts over a run of 10000 occurrences against twice 1024: four groups in flight took 1.9 times as long, one takes as long."""
    import time

    import torch

    import paper_2408_05676_amd as laser
    rng = np.random.default_rng(0)
    trunk, count, K = rng.integers(8, 30000, 40), 10000, 16
    text = np.tile(np.concatenate([[7], trunk]), (count, 1))
    hit = rng.random(text.shape) < 0.1
    hit[:, 0] = False
    text[hit] = rng.integers(8, 30000, int(hit.sum()))
    pool = laser.Pool(text.reshape(-1).astype(np.int32), np.arange(count + 1, dtype=np.int64) * 41, np.zeros(count, np.int64), 2)
    took = []
    for B in (1024, 2048):
        i32 = dict(dtype=torch.int32, device="cuda")
        qk, tail = torch.zeros(B, dtype=torch.int64, device="cuda"), torch.tensor([[1, 7]] * B, **i32)
        out = (torch.empty((B, K), **i32), torch.empty(B, **i32), torch.empty(B, **i32), torch.empty(B, dtype=torch.int64, device="cuda"))
        best = 1e9
        for _ in range(5):
            torch.cuda.synchronize()
            t = time.perf_counter()
            laser.retrieve_drafts(pool, qk, tail, 1, 2, K, 1, out=out)
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t)
        took.append(best)
    pool.close()
    assert took[1] <= 1.5 * took[0], took
