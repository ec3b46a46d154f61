"""Pools on both sides of the size from which their index is built on the device: lookups, tokens and the number of
index entries against oracle.retrieval, exactly."""
import numpy as np
import pytest
import torch

from oracle.retrieval import RegroupedPool, retrieve

pytestmark = pytest.mark.gpu

HOST_MAX = 4095          # occurrences (tokens minus sequences) up to which the host builds


def _texts(rng, lens, vocab):
    toks = rng.integers(0, vocab, int(np.sum(lens))).astype(np.int32)
    return toks, np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)


def _entries(src, n_max):
    """Distinct (key, n, n-gram) that have a successor in their sequence."""
    n_runs = 0
    for seqs in _sequences(src).values():
        grams = [set() for _ in range(n_max)]
        for s in seqs:
            for n in range(1, n_max + 1):
                for e in range(n - 1, len(s) - 1):
                    grams[n - 1].add(s[e - n + 1:e + 1])
        n_runs += sum(len(g) for g in grams)
    return n_runs


def _sequences(src):
    toks, off, keys = src
    out = {}
    for i, k in enumerate(keys.tolist()):
        out.setdefault(k, []).append(tuple(toks[off[i]:off[i + 1]].tolist()))
    return out


def _check(toks, off, keys, n_max, seed, K=6):
    import paper_2408_05676_amd as laser
    rng = np.random.default_rng(seed)
    pool = laser.Pool(toks, off, keys, n_max)
    ora = RegroupedPool(toks, off, keys)
    info = pool.info()
    assert info["n_tokens"] == toks.size and info["n_keys"] == np.unique(keys).size
    assert info["n_index_entries"] == _entries((toks, off, keys), n_max)
    assert (pool.read_tokens(0, toks.size) == ora.P).all()
    # contexts that occur, contexts that do not, keys that do not
    B = 96
    at = rng.integers(0, toks.size - n_max, B)
    tails = np.stack([toks[a:a + n_max] for a in at]).astype(np.int32)
    seq = np.searchsorted(off, at, side="right") - 1
    qk = keys[seq].copy()
    qk[::11] = 1 << 50
    tails[::7] = rng.integers(0, int(toks.max()) + 1, tails[::7].shape)
    tails[::13, 0] = -1
    g = laser.retrieve_drafts(pool, torch.tensor(qk, device="cuda"), torch.tensor(tails, device="cuda"), 1, n_max, K, 1)
    got = [t.cpu().numpy() for t in g]
    want = retrieve(ora, qk, tails, 1, n_max, K, 1)
    for name, x, y in zip(("drafts", "draft_len", "match_n", "pool_index"), got, want):
        assert (x == y).all(), name
    pool.close()


@pytest.mark.parametrize("n_sa", [HOST_MAX, HOST_MAX + 1, 4 * 4096, 4 * 4096 + 1, 10 * 2048 - 1])
def test_sizes_around_the_rule_and_the_tiles(n_sa):
    rng = np.random.default_rng(n_sa)
    lens = np.full(200, 1)
    lens += rng.multinomial(n_sa, np.ones(200) / 200)           # one successor fewer than tokens in each
    toks, off = _texts(rng, lens, 50)
    _check(toks, off, rng.integers(-3, 4, 200).astype(np.int64) * 1000003, 3, n_sa)


@pytest.mark.parametrize("vocab,n_max", [(1, 2), (2, 8), (255, 1), (256, 3), (65535, 2), (70000, 4), (2**31 - 1, 2)])
def test_token_widths_and_ngrams(vocab, n_max):
    """Digits of one to four bytes; runs that span many workgroups (vocab 1, 2) and runs of one."""
    rng = np.random.default_rng(vocab % 1000)
    lens = rng.integers(0, 120, 500)                            # empty and one-token sequences among them
    toks, off = _texts(rng, lens, vocab)
    if vocab > 1000:                                            # the largest ids, and some that repeat
        toks[rng.random(toks.size) < 0.5] = vocab - 1
    _check(toks, off, rng.integers(0, 5, 500).astype(np.int64), n_max, vocab % 1000, K=3)


@pytest.mark.parametrize("vocab", [65535, 65536, 2**31 - 1])
@pytest.mark.parametrize("n_sa", [4095, 4096, 8191, 8192])
def test_sizes_around_the_rule_by_token_width(n_sa, vocab):
    """Tokens of more than two bytes go to the device from twice the size on."""
    rng = np.random.default_rng(n_sa + vocab % 1000)
    lens = np.full(100, 1)
    lens += rng.multinomial(n_sa, np.ones(100) / 100)
    toks, off = _texts(rng, lens, vocab)
    toks[rng.random(toks.size) < 0.4] = vocab - 1
    toks[0] = vocab - 1
    _check(toks, off, rng.integers(0, 3, 100).astype(np.int64), 3, n_sa)


@pytest.mark.parametrize("n_keys", [1, 255, 257, 9000])
def test_sub_pools(n_keys):
    rng = np.random.default_rng(n_keys)
    lens = rng.integers(1, 5, 12000)
    lens[0] = 9000
    toks, off = _texts(rng, lens, 12)
    _check(toks, off, (rng.integers(0, n_keys, 12000) * 7919 - 5000).astype(np.int64), 4, n_keys)


def test_refusals_stay():
    import paper_2408_05676_amd as laser
    toks = np.ones(40000, np.int32)
    toks[30001] = -1
    off = np.array([0, 20000, 40000], np.int64)
    with pytest.raises(laser.LaserError, match="negative token in sequence 1"):
        laser.Pool(toks, off, np.zeros(2, np.int64), 3)
    with pytest.raises(laser.LaserError, match="not ascending"):
        laser.Pool(np.ones(40000, np.int32), np.array([0, 41000, 40000], np.int64), np.zeros(2, np.int64), 3)


def test_a_build_does_not_wait_for_other_streams_and_keeps_no_working_memory():
    """The working arrays (20 MiB here) are allocated and given back in the order of the caller's stream: the build ends while another
    stream is still at work, and only the pool's own memory stays taken."""
    import paper_2408_05676_amd as laser
    rng = np.random.default_rng(2)
    lens = np.full(10000, 120)
    toks, off = _texts(rng, lens, 32000)
    keys = rng.integers(0, 50, 10000).astype(np.int64)
    laser.Pool(toks, off, keys, 2).close()                      # first use of the kernels
    other = torch.cuda.Stream()
    with torch.cuda.stream(other):
        torch.cuda._sleep(1)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    with torch.cuda.stream(other):
        torch.cuda._sleep(1_000_000_000)                        # some hundred ms on one compute unit
    pool = laser.Pool(toks, off, keys, 2)
    assert not other.query(), "the build waited for the other stream"
    taken = free - torch.cuda.mem_get_info()[0]
    assert taken <= pool.info()["device_bytes"] + (12 << 20), taken    # (allocations are rounded up to 2 MiB)
    torch.cuda.synchronize()
    pool.close()


def _everything(pool, toks, keys, n_max):
    """Counts, tokens, and lookups of all kinds of contexts in a pool."""
    import paper_2408_05676_amd as laser
    rng = np.random.default_rng(1)
    at = rng.integers(0, toks.size - n_max, 300)
    tails = np.stack([toks[a:a + n_max] for a in at]).astype(np.int32)
    tails[::5] = rng.integers(0, int(toks.max()) + 1, tails[::5].shape)
    qk = keys[rng.integers(0, keys.size, 300)]
    dev = [torch.tensor(x, device="cuda") for x in (qk, tails)]
    found = [t.cpu().numpy() for t in laser.retrieve_drafts(pool, *dev, 1, n_max, 9, 1)]
    return [np.array(sorted(pool.info().items())), pool.read_tokens(0, toks.size)] + found


# The pool and the working arrays in the order in which they are allocated: the tokens, their ends, the occurrences, the
# working arrays, and after the kernels the table.
@pytest.mark.parametrize("share", [0.0, 0.3, 0.5, 0.9, 0.999])
def test_a_build_that_finds_no_memory_goes_on_on_the_host(share):
    import paper_2408_05676_amd as laser
    rng = np.random.default_rng(7)
    lens = rng.integers(0, 90, 700)
    toks, off = _texts(rng, lens, 40)
    keys = rng.integers(0, 9, 700).astype(np.int64)
    host = laser.Pool(toks, off, keys, 3, builder="host")
    want = _everything(host, toks, keys, 3)
    whole = laser.Pool(toks, off, keys, 3, builder="device")
    n_blk = -(-toks.size // 4096)
    work = 17 * toks.size + 1024 * n_blk                        # at least; the pool's own arrays come on top
    limit = int(share * (whole.info()["device_bytes"] + work))
    short = laser.Pool(toks, off, keys, 3, mem_limit=limit)
    for pool in (whole, short):
        for x, y in zip(_everything(pool, toks, keys, 3), want):
            assert (x == y).all()
    for pool in (host, whole, short):
        pool.close()


@pytest.mark.parametrize("builder", ["host", "device"])
@pytest.mark.parametrize("lens", [[2], [0, 3, 1, 0], [1, 1], [5000], [70] * 100])
def test_either_builder_takes_any_size(builder, lens):
    import paper_2408_05676_amd as laser
    rng = np.random.default_rng(len(lens))
    toks, off = _texts(rng, lens, 6)
    keys = rng.integers(0, 2, len(lens)).astype(np.int64)
    pool, ora = laser.Pool(toks, off, keys, 2, builder=builder), RegroupedPool(toks, off, keys)
    assert pool.info()["n_index_entries"] == _entries((toks, off, keys), 2)
    qk, tails = np.repeat(keys[:1], 36), np.array([[a, b] for a in range(6) for b in range(6)], np.int32)
    got = laser.retrieve_drafts(pool, torch.tensor(qk, device="cuda"), torch.tensor(tails, device="cuda"), 1, 2, 4, 1)
    for x, y in zip(got, retrieve(ora, qk, tails, 1, 2, 4, 1)):
        assert (x.cpu().numpy() == y).all()
    pool.close()
