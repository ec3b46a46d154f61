"""The work a user of this library has it do, as measurable cases over the public entry points.

Six kinds of case, all built from a seed alone:

  step      one decoding step of a running batch: retrieve drafts (chain or token tree) -> verify -> commit -> context update
  prefill   prompts of a batch into an empty cache through Engine.prefill, then the first one-row step
  generate  laser_generate: the whole text of a batch, with or without the sequences' own text as a temporary branch
  head      the output head + relaxed acceptance alone, at a large vocabulary
  retrieve  a batch of draft lookups (chains, chains with a temporary branch, or token trees)
  build     a retrieval pool from host arrays, and a batch of lookups in it

Model shapes, pool shapes, batch sizes, context lengths and draft lengths are those of this repository's benchmark
workloads and tests, spread over the ranges between them. Weights are random, with one structure laid over them: the
output head holds, for every token, the direction of the token before it on one long cycle over the vocabulary, so that
the model follows that cycle with confidence, as a trained model follows a text its pool already holds. Pool texts are
noisy pieces of the cycle: drafts are accepted in runs that break where a pool text was substituted.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2408_05676_amd as laser
from paper_2408_05676_amd.harness import Engine

LM_GAIN = 5.0          # final-norm gain: sharp enough that the acceptance threshold p = 0.1 separates
PRM = dict(topk=2, p=0.1)


class Shape:
    """Decoder shape as the Engine wants it."""

    def __init__(self, n_layers, d, n_heads, ffn, vocab):
        self.n_layers, self.d, self.n_heads, self.ffn, self.vocab = n_layers, d, n_heads, ffn, vocab
        self.head_dim, self.eps, self.rope_base = d // n_heads, 1e-6, 10000.0

    def streamed_params(self):
        return self.n_layers * (4 * self.d * self.d + 3 * self.d * self.ffn) + self.vocab * self.d


SHAPES = {
    "tiny": Shape(2, 256, 4, 1024, 2048),
    "1b": Shape(16, 2048, 16, 5632, 32000),
    "7b": Shape(32, 4096, 32, 11008, 32000),
}


def listed():
    return [
        # smallest calls: a two-layer model, where launches and host work are all there is
        dict(name="step_tiny_b2_k4", kind="step", shape="tiny", B=2, ctx=64, K=4, tree=False, pool="tiny", mode=0),
        # the latency workload: one user, a 7B model, chains of 8
        dict(name="step_7b_b1_k8", kind="step", shape="7b", B=1, ctx=1024, K=8, tree=False, pool="latency", mode=0),
        # plain decoding without drafts: four running sequences, one row each
        dict(name="decode_1b_b4_k0", kind="step", shape="1b", B=4, ctx=700, K=0, tree=False, pool="tiny", mode=0),
        # small batches, 72 rows
        dict(name="step_1b_b8_k8", kind="step", shape="1b", B=8, ctx=512, K=8, tree=False, pool="keyed", mode=0),
        dict(name="step_7b_b8_k8", kind="step", shape="7b", B=8, ctx=1024, K=8, tree=False, pool="latency", mode=1),
        # the throughput workload: 64 users, chains of 10, 704 rows
        dict(name="step_7b_b64_k10", kind="step", shape="7b", B=64, ctx=512, K=10, tree=False, pool="zipf", mode=0),
        # token trees of 16 nodes, 136 rows
        dict(name="tree_1b_b8_k16", kind="step", shape="1b", B=8, ctx=333, K=16, tree=True, pool="keyed", mode=0),
        # prompts into the cache, 256 rows per forward
        dict(name="prefill_7b_b4", kind="prefill", shape="7b", B=4, ctx=500, chunk=64),
        # the output head at a 128 k vocabulary
        dict(name="head_128k_b64_k15", kind="head", vocab=128256, d=4096, B=64, K=15, mode=0),
        # many users' lookups at once
        dict(name="retrieve_b4096_k16", kind="retrieve", pool="zipf", B=4096, K=16, n_max=4, form="chain"),
        # a pool of one million tokens from host arrays
        dict(name="build_1m", kind="build", n_seq=3906, seq_len=256, n_keys=10000, n_max=3),
        # whole texts with the temporary branch
        dict(name="generate_1b_b8", kind="generate", shape="1b", B=8, ctx=96, K=8, tree=False, own=True, max_new=48, mode=0),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "step", "prefill", "generate", "head", "retrieve", "build"])
    if kind == "step":
        shape = rng.choice(["tiny", "1b", "1b", "7b", "7b"])
        tree = rng.random() < 0.25
        K = rng.randint(2, 16) if tree else rng.choice([0, rng.randint(1, 10), rng.randint(4, 16)])
        B = _log_int(rng, 1, 64)
        # no more rows than the largest listed step at the same width
        B = max(1, min(B, 704 // (K + 1)))
        pool = rng.choice(["tiny"] if shape == "tiny" else ["latency", "keyed", "zipf"])
        return dict(kind="step", shape=shape, B=B, ctx=_log_int(rng, 40, 1024 if B < 32 else 512), K=K, tree=tree and K > 0, pool=pool,
                    mode=rng.randint(0, 3))
    if kind == "prefill":
        shape = rng.choice(["tiny", "1b", "7b"])
        B, chunk = _log_int(rng, 1, 16), rng.choice([16, 33, 64])
        # no more forwards and no more tokens than the listed prompts take
        return dict(kind="prefill", shape=shape, B=B, ctx=_log_int(rng, 40, min(1984 // B, 8 * chunk)), chunk=chunk)
    if kind == "generate":
        tree = rng.random() < 0.4
        return dict(kind="generate", shape=rng.choice(["tiny", "1b"]), B=_log_int(rng, 1, 12), ctx=_log_int(rng, 20, 200), K=rng.randint(2, 12),
                    tree=tree, own=not tree and rng.random() < 0.6, max_new=rng.randint(12, 48), mode=rng.randint(0, 3))
    if kind == "head":
        K = rng.randint(0, 20)
        vocab = rng.choice([32000, 50272, 128256])
        B = max(1, min(_log_int(rng, 1, 64), 1024 // (K + 1)))
        return dict(kind="head", vocab=vocab, d=rng.choice([2048, 4096]), B=B, K=K, mode=rng.randint(0, 3))
    if kind == "retrieve":
        form = rng.choice(["chain", "chain", "own", "tree"])
        return dict(kind="retrieve", pool=rng.choice(["latency", "keyed", "zipf"]), B=_log_int(rng, 1, 16384 if form == "chain" else 1024),
                    K=rng.randint(1, 32), n_max=rng.randint(2, 4), form=form)
    return dict(kind="build", n_seq=_log_int(rng, 10, 3906), seq_len=rng.randint(20, 256), n_keys=_log_int(rng, 1, 10000), n_max=rng.randint(1, 4))


# ------------------------------------------------------------------------------------------------ texts and pools
POOLS = {
    #            texts, length, templates, keys, zipf
    "tiny": dict(n_seq=500, seq_len=64, n_templ=20, n_keys=1, zipf=False),
    "latency": dict(n_seq=2000, seq_len=256, n_templ=50, n_keys=1, zipf=False),
    "keyed": dict(n_seq=3000, seq_len=256, n_templ=200, n_keys=300, zipf=False),
    "zipf": dict(n_seq=3906, seq_len=256, n_templ=500, n_keys=10000, zipf=True),
}
SUB_RATE = 0.10        # share of a pool text's tokens that differ from the text the model would write


def make_texts(rng, cycle, n_seq, seq_len, n_templ, n_keys, zipf):
    """Pool texts: noisy pieces of the cycle, two templates per key, lengths between half of seq_len and seq_len."""
    vocab = cycle.size
    if zipf:
        w = np.arange(1, n_keys + 1, dtype=np.float64) ** -1.1
        rank = np.searchsorted(np.cumsum(w) / w.sum(), rng.random(n_seq), side="right").clip(max=n_keys - 1)
    else:
        rank = np.arange(n_seq) % n_keys
    start = rng.integers(0, vocab, n_templ)
    templ = (rank * 7 + rng.integers(0, 2, n_seq)) % n_templ
    low = max(2, seq_len // 2)
    length = rng.permutation(low + np.arange(n_seq) % (seq_len + 1 - low))
    off = np.zeros(n_seq + 1, dtype=np.int64)
    np.cumsum(length, out=off[1:])
    seq = np.repeat(np.arange(n_seq), length)
    pos = np.arange(off[-1]) - off[seq]
    tokens = cycle[(start[templ[seq]] + pos) % vocab].astype(np.int32)
    hit = rng.random(tokens.size) < SUB_RATE
    tokens[hit] = rng.integers(0, vocab, int(hit.sum()))
    key = (rank.astype(np.int64) * 2654435761 + 12345) % (1 << 40)
    return dict(tokens=tokens, off=off, key=key, start=start[templ], length=length)


def pick_contexts(rng, texts, B, room):
    """B running texts of the pool's keys: (key, place on the cycle) with `room` template tokens still ahead where it is long enough."""
    s = rng.integers(0, texts["key"].size, B)
    cut = 4 + (rng.random(B) * np.maximum(texts["length"][s] - room - 4, 1)).astype(np.int64)
    return texts["key"][s], texts["start"][s] + cut


def cuda(a, dtype=None):
    t = torch.from_numpy(np.ascontiguousarray(a))
    return (t if dtype is None else t.to(dtype)).cuda()


# ------------------------------------------------------------------------------------------------ models
def make_weights(sh, gen, cycle):
    def mat(*dims, std=0.02):
        return torch.empty(dims, dtype=torch.bfloat16, device="cuda").normal_(0.0, std, generator=gen)

    def gain(*dims):
        return torch.empty(dims, dtype=torch.float32, device="cuda").normal_(1.0, 0.1, generator=gen)

    L, d, F, V = sh.n_layers, sh.d, sh.ffn, sh.vocab
    # the residual stream of the layers has about this size at random weights of standard deviation 0.02; embeddings of
    # 1.5 times that keep the current token's direction in the final state
    s = 0.02 * math.sqrt(d)
    emb_std = 1.5 * 0.02 * math.sqrt(F) * 0.55 * s * s * math.sqrt(L)
    w = {"wqkv": mat(L, 3 * d, d), "wo": mat(L, d, d), "wgu": mat(L, 2 * F, d), "wdown": mat(L, d, F), "g1": gain(L, d), "g2": gain(L, d),
         "emb": mat(V, d, std=emb_std), "wlm": mat(V, d), "gf": gain(d) * LM_GAIN}
    here = cuda(cycle, torch.int64)
    w["wlm"][here.roll(-1)] += (w["emb"][here].float() * (0.229 / (math.sqrt(d) * emb_std))).to(torch.bfloat16)
    return w


def make_engine(sh, seed, B, K, max_len, cycle, **kw):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    return Engine(sh, make_weights(sh, gen, cycle), B, K, max_len, **kw), gen


def fill_cache(eng, gen, lens):
    """Caches of the given lengths with keys and values of the sizes the layers produce (from another worker, say)."""
    sh = eng.shape
    for layer in range(sh.n_layers):
        for s, t in enumerate(lens):
            kv = torch.empty((2, int(t), sh.n_heads, sh.head_dim), dtype=torch.float16, device="cuda").normal_(0.0, 1.28, generator=gen)
            eng.kv.import_layer(s, layer, kv[0], kv[1])


def prepare(case, seed):
    rng = np.random.default_rng(seed)
    return {"step": _prep_step, "prefill": _prep_prefill, "generate": _prep_generate, "head": _prep_head, "retrieve": _prep_retrieve,
            "build": _prep_build}[case["kind"]](case, seed, rng)


def run(state):
    return state["run"](state)


# ------------------------------------------------------------------------------------------------ step
def _prep_step(case, seed, rng):
    sh, B, K = SHAPES[case["shape"]], case["B"], case["K"]
    cycle = rng.permutation(sh.vocab)
    texts = make_texts(rng, cycle, **POOLS[case["pool"]])
    key, place = pick_contexts(rng, texts, B, K + 4)
    # running sequences have different lengths: the named context is the longest
    lens = case["ctx"] - rng.integers(0, max(1, case["ctx"] // 4), B)
    lens[0] = case["ctx"]
    eng, gen = make_engine(sh, seed, B, K, case["ctx"] + K + 17, cycle)
    fill_cache(eng, gen, lens - 1)
    tail = cycle[(place[:, None] + np.arange(-eng.n_max, 0)) % sh.vocab].astype(np.int32)
    pool = laser.Pool(texts["tokens"], texts["off"], texts["key"], eng.n_max)
    eng.set_pool(pool, key)
    st = dict(run=_run_tree if case["tree"] else _run_step, eng=eng, pool=pool, lens=[int(t) - 1 for t in lens], tail=cuda(tail),
              pending=cuda(tail[:, -1]), mode=case["mode"], K=K)
    if case["tree"]:
        i32 = dict(dtype=torch.int32, device="cuda")
        st["tree"] = (torch.empty((B, K), **i32), torch.empty((B, K), **i32), None, torch.empty(B, **i32), torch.empty(B, **i32))
    return st


def _run_step(st):
    eng = st["eng"]
    for s, n in enumerate(st["lens"]):
        eng.kv.set_len(s, n)
    tail, pending = st["tail"].clone(), st["pending"].clone()
    if st["K"] > 0:
        laser.retrieve_drafts(st["pool"], eng.keys, tail, 1, eng.n_max, st["K"], 1, out=(eng.drafts, eng.draft_len, eng.match_n, eng.pool_index))
    acc, out, logits = laser.verify_step(eng.model, eng.kv, eng.seq_ids, pending, eng.drafts, eng.draft_len, PRM["topk"], PRM["p"], st["mode"],
                                         want_logits=True)
    laser.kv_commit(eng.kv, eng.seq_ids, acc)
    laser.ctx_advance(tail, pending, out, acc)
    return eng.drafts, eng.draft_len, acc, out, logits, tail, pending


def _run_tree(st):
    eng = st["eng"]
    for s, n in enumerate(st["lens"]):
        eng.kv.set_len(s, n)
    tail, pending = st["tail"].clone(), st["pending"].clone()
    tok, par, _, tl, _ = laser.retrieve_tree(st["pool"], eng.keys, tail, 1, eng.n_max, st["K"], 1, out=st["tree"])
    acc, out, path, logits = laser.verify_tree(eng.model, eng.kv, eng.seq_ids, pending, tok, par, tl, PRM["topk"], PRM["p"], st["mode"],
                                               want_logits=True)
    laser.kv_commit_tree(eng.kv, eng.seq_ids, acc, path)
    laser.ctx_advance(tail, pending, out, acc)
    return tok, par, tl, acc, out, path, logits, tail, pending


# ------------------------------------------------------------------------------------------------ prefill
def _prep_prefill(case, seed, rng):
    sh, B = SHAPES[case["shape"]], case["B"]
    cycle = rng.permutation(sh.vocab)
    eng, _ = make_engine(sh, seed, B, 0, case["ctx"] + 17, cycle, prefill_chunk=case["chunk"])
    prompts = cycle[(rng.integers(0, sh.vocab, (B, 1)) + np.arange(case["ctx"])) % sh.vocab].astype(np.int32)
    hit = rng.random(prompts.shape) < 0.3
    prompts[hit] = rng.integers(0, sh.vocab, int(hit.sum()))
    return dict(run=_run_prefill, eng=eng, prompts=prompts)


def _run_prefill(st):
    eng = st["eng"]
    for s in range(eng.B):
        eng.kv.set_len(s, 0)
    eng.prefill(st["prompts"])
    acc, out, logits = laser.verify_step(eng.model, eng.kv, eng.seq_ids, eng.pending, eng.drafts, eng.draft_len, 1, -1.0, want_logits=True)
    return acc, out, logits


# ------------------------------------------------------------------------------------------------ generate
def _prep_generate(case, seed, rng):
    sh, B, K = SHAPES[case["shape"]], case["B"], case["K"]
    cycle = rng.permutation(sh.vocab)
    texts = make_texts(rng, cycle, **POOLS["tiny" if case["shape"] == "tiny" else "keyed"])
    key, place = pick_contexts(rng, texts, B, case["max_new"])
    eng, gen = make_engine(sh, seed, B, K, case["ctx"] + case["max_new"] + K + 17, cycle)
    fill_cache(eng, gen, [case["ctx"] - 1] * B)
    ctx = cycle[(place[:, None] + np.arange(-case["ctx"], 0)) % sh.vocab].astype(np.int32)
    pool = laser.Pool(texts["tokens"], texts["off"], texts["key"], eng.n_max)
    eng.set_pool(pool, key)
    st = dict(run=_run_generate, eng=eng, pool=pool, case=case, tail=cuda(ctx[:, -eng.n_max:]), pending=cuda(ctx[:, -1]),
              none=torch.empty((B, 0), dtype=torch.int32, device="cuda"), zero=torch.zeros(B, dtype=torch.int32, device="cuda"))
    if case["own"]:
        own = np.zeros((B, case["ctx"] + case["max_new"] + K + 1), dtype=np.int32)
        own[:, :case["ctx"]] = ctx
        st["own"], st["own_len"] = cuda(own), torch.full((B,), case["ctx"], dtype=torch.int32, device="cuda")
    return st


def _run_generate(st):
    eng, c = st["eng"], st["case"]
    for s in range(eng.B):
        eng.kv.set_len(s, c["ctx"] - 1)
    own = dict(own_tokens=st["own"].clone(), own_len=st["own_len"].clone()) if c["own"] else {}
    pending = st["pending"].clone()
    gen, n, cnt, steps, _ = laser.generate(eng.model, eng.kv, st["pool"], eng.seq_ids, eng.keys, st["tail"].clone(), pending, c["K"], 1,
                                           PRM["topk"], PRM["p"], c["mode"], max_new_tokens=c["max_new"], tree=c["tree"], **own)
    # the distribution that the next token would come from
    acc, out, logits = laser.verify_step(eng.model, eng.kv, eng.seq_ids, pending, st["none"], st["zero"], 1, -1.0, want_logits=True)
    return gen, n, cnt, out, logits


# ------------------------------------------------------------------------------------------------ head
def _prep_head(case, seed, rng):
    V, d, B, K = case["vocab"], case["d"], case["B"], case["K"]
    gen = torch.Generator(device="cuda").manual_seed(seed)
    w = torch.empty((V, d), dtype=torch.bfloat16, device="cuda").normal_(0.0, 0.02, generator=gen)
    model = laser.Model(0, d, d // 128, 128, V, {"wlm": w}, B * (K + 1), B, 0)
    # hidden states along the direction of one vocabulary entry, from unsure to sure, so that drafts lie on both sides of
    # the threshold; an eighth of the drafts name another token
    planted = cuda(rng.integers(0, V, (B, K + 1)))
    noise = torch.empty((B, K + 1, d), device="cuda").normal_(0.0, 0.5, generator=gen)
    amp = cuda((4096.0 / d) * (5.0 + 9.0 * rng.random((B, K + 1, 1))), torch.float32)
    h = (amp * w[planted].float() + noise).to(torch.float16)
    drafts = planted[:, :K].to(torch.int32).cpu().numpy()
    wrong = rng.random(drafts.shape) < 0.125
    drafts[wrong] = rng.integers(0, V, int(wrong.sum()))
    return dict(run=_run_head, model=model, h=h, drafts=cuda(drafts), n=torch.full((B,), K, dtype=torch.int32, device="cuda"), mode=case["mode"])


def _run_head(st):
    return laser.verify_head(st["model"], st["h"], st["drafts"], st["n"], PRM["topk"], PRM["p"], st["mode"], want_logits=True)


# ------------------------------------------------------------------------------------------------ retrieve
OWN_CAP = 512


def _prep_retrieve(case, seed, rng):
    vocab, B, n_max, K = 32000, case["B"], case["n_max"], case["K"]
    cycle = rng.permutation(vocab)
    texts = make_texts(rng, cycle, **POOLS[case["pool"]])
    pool = laser.Pool(texts["tokens"], texts["off"], texts["key"], n_max)
    key, place = pick_contexts(rng, texts, B, K)
    ctx = cycle[(place[:, None] + np.arange(-OWN_CAP, 0)) % vocab].astype(np.int32)
    hit = rng.random(ctx.shape) < SUB_RATE
    ctx[hit] = rng.integers(0, vocab, int(hit.sum()))
    new = rng.random(B) < 0.05                     # users without a pool
    key = np.where(new, -1 - np.arange(B), key)
    i32 = dict(dtype=torch.int32, device="cuda")
    st = dict(run=_run_retrieve, pool=pool, case=case, keys=cuda(key), tail=cuda(ctx[:, -n_max:]))
    if case["form"] == "tree":
        st["out"] = (torch.empty((B, K), **i32), torch.empty((B, K), **i32), torch.empty((B, K), **i32), torch.empty(B, **i32), torch.empty(B, **i32))
    else:
        st["out"] = (torch.empty((B, K), **i32), torch.empty(B, **i32), torch.empty(B, **i32), torch.empty(B, dtype=torch.int64, device="cuda"))
    if case["form"] == "own":
        st["own"], st["own_len"] = cuda(ctx), cuda(rng.integers(n_max, OWN_CAP + 1, B).astype(np.int32))
    return st


def _run_retrieve(st):
    c = st["case"]
    if c["form"] == "tree":
        return laser.retrieve_tree(st["pool"], st["keys"], st["tail"], 1, c["n_max"], c["K"], 1, out=st["out"])
    if c["form"] == "own":
        return laser.retrieve_drafts_temp(st["pool"], st["keys"], st["tail"], st["own"], st["own_len"], 1, c["n_max"], c["K"], 1, out=st["out"])
    return laser.retrieve_drafts(st["pool"], st["keys"], st["tail"], 1, c["n_max"], c["K"], 1, out=st["out"])


# ------------------------------------------------------------------------------------------------ build
def _prep_build(case, seed, rng):
    vocab = 32000
    cycle = rng.permutation(vocab)
    texts = make_texts(rng, cycle, n_seq=case["n_seq"], seq_len=case["seq_len"], n_templ=max(1, case["n_seq"] // 8), n_keys=case["n_keys"],
                       zipf=case["n_keys"] > 1)
    key, place = pick_contexts(rng, texts, 256, 8)
    tail = cycle[(place[:, None] + np.arange(-case["n_max"], 0)) % vocab].astype(np.int32)
    return dict(run=_run_build, texts=texts, n_max=case["n_max"], keys=cuda(key), tail=cuda(tail))


def _run_build(st):
    t = st["texts"]
    pool = laser.Pool(t["tokens"], t["off"], t["key"], st["n_max"])
    info = pool.info()
    found = laser.retrieve_drafts(pool, st["keys"], st["tail"], 1, st["n_max"], 8, 1)
    out = (np.array([info["n_tokens"], info["n_keys"], info["n_index_entries"]]), pool.read_tokens(0, info["n_tokens"]), *found)
    pool.close()
    return out


# ------------------------------------------------------------------------------------------------ work and tolerance
def _forward_work(sh, rows, ctx_tokens, row_ctx):
    """One forward over `rows` rows: streamed weights once, the cached keys and values (5 bytes per element pair, the
    documented cache format) of `ctx_tokens` tokens once, the rows' own keys and values written; products of the rows
    with the weights and of each row with its context (`row_ctx` row-token pairs)."""
    kv = 5 * sh.n_layers * sh.d
    return dict(bytes=2 * sh.streamed_params() + kv * (ctx_tokens + rows), flops=2 * rows * sh.streamed_params() + 4 * sh.n_layers * sh.d * row_ctx)


def work(case):
    kind = case["kind"]
    if kind == "step":
        sh, B, R = SHAPES[case["shape"]], case["B"], case["K"] + 1
        ctx = int(case["ctx"] * (1.0 if B == 1 else 0.875))          # the mean of the lengths drawn
        w = _forward_work(sh, B * R, B * ctx, B * R * ctx)
        w["bytes"] += 4 * B * R * sh.vocab                           # logits
        return w
    if kind == "prefill":
        sh, B, T = SHAPES[case["shape"]], case["B"], case["ctx"] - 1
        n_fwd = math.ceil(T / case["chunk"])
        # a forward reads what earlier ones cached; the last step reads everything and writes its logits
        w = _forward_work(sh, 0, 0, 0)
        head = sh.vocab * sh.d
        rows = B * T
        body = sh.streamed_params() - head
        return dict(bytes=n_fwd * 2 * body + w["bytes"] + 5 * sh.n_layers * sh.d * (B * T * (n_fwd - 1) // 2 + 2 * B * T) + 4 * B * sh.vocab,
                    flops=2 * rows * body + 4 * sh.n_layers * sh.d * B * T * T // 2 + 2 * B * sh.streamed_params())
    if kind == "generate":
        sh, B, R = SHAPES[case["shape"]], case["B"], case["K"] + 1
        n = max(2, round(case["max_new"] / min(5.0, R)))             # steps, with about four drafts accepted in each
        one = _forward_work(sh, B * R, B * (case["ctx"] + case["max_new"] // 2), B * R * (case["ctx"] + case["max_new"] // 2))
        last = _forward_work(sh, B, B * (case["ctx"] + case["max_new"]), B * (case["ctx"] + case["max_new"]))
        return dict(bytes=n * one["bytes"] + last["bytes"] + 4 * B * sh.vocab, flops=n * one["flops"] + last["flops"])
    if kind == "head":
        rows = case["B"] * (case["K"] + 1)
        return dict(bytes=2 * case["vocab"] * case["d"] + 2 * rows * case["d"] + 4 * rows * case["vocab"], flops=2 * rows * case["vocab"] * case["d"])
    if kind == "retrieve":
        B, K = case["B"], case["K"]
        # a probe per context, a few dozen occurrences and their successors, the results
        return dict(bytes=B * (8 + 4 * case["n_max"] + 16 + 32 * (8 + 4 * min(K, 8)) + 4 * K + 16 + (2 * OWN_CAP if case["form"] == "own" else 0)), flops=0)
    n = case["n_seq"] * case["seq_len"] * 3 // 4
    # tokens in; tokens, sequence ends, occurrence array and a half-full table of the distinct n-grams out
    return dict(bytes=n * (4 + 4 + 4 + 4) + 32 * n * case["n_max"] // 2, flops=0)


def tolerance(case):
    # Lookups and pools are exact. Logits: activations are rounded to fp16 at several points of every layer, so another
    # order of the sums moves the roundings: measured between the library's own kernel choices for one step (persistent
    # or per-operation kernels, context split or whole, reductions in one or several parts, one or two activation
    # planes) 2.4e-4 .. 4.1e-4; the head alone, against a float32 product of the same operands, 1.0e-6. Four times that.
    # The model is sure of its next token, so tokens and accepted lengths do not move with the last bits; at the head a
    # draft may sit on the threshold.
    if case["kind"] in ("retrieve", "build"):
        return "exact"
    if case["kind"] == "head":
        return {"rel": 4e-6, "max": 2.7e-4, "differ": 0.01}
    return {"rel": 1.6e-3, "differ": 0.001}
