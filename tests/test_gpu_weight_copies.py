"""Which weights a call reads -- the caller's matrices or the fp16 copies the handle makes of them -- and how long the copies' memory lives."""
import pytest
import torch

import synth
from tests import gpu_util as gu


pytestmark = pytest.mark.gpu


def _head(d, V, rows, seed=1):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    w = torch.empty((V, d), dtype=torch.bfloat16, device="cuda").normal_(0.0, 0.1, generator=gen)
    h = torch.empty((1, rows, d), dtype=torch.float16, device="cuda").normal_(generator=gen)
    return w, h, torch.zeros((1, rows - 1), dtype=torch.int32, device="cuda"), torch.full((1,), rows - 1, dtype=torch.int32, device="cuda")


@pytest.mark.parametrize("topk", [2, 5])
@pytest.mark.parametrize("rows", [16, 17, 24, 64])
def test_the_head_alone_reads_the_callers_matrix(rows, topk):
    """Up to 80 rows at every call: a matrix changed in place between two calls is seen by the second, which makes no copy."""
    import paper_2408_05676_amd as laser
    d, V = 1024, 32768                                                    # a copy would take 64 MB
    w, h, drafts, n = _head(d, V, rows)
    model = laser.Model(0, d, 8, 128, V, {"wlm": w}, rows, 1, 0)
    for turn in range(2):
        free = torch.cuda.mem_get_info()[0]
        logits = laser.verify_head(model, h, drafts, n, topk, -1.0, 2, want_logits=True)[2]
        torch.cuda.synchronize()
        # (torch itself takes blocks of at most 20 MB for the results)
        assert free - torch.cuda.mem_get_info()[0] < 48 << 20
        want = h[0].double() @ w.double().t()
        # products of fp16 and bf16 are exact in float32, 1024 of them are added in float32
        assert float((logits[0].double() - want).norm() / want.norm()) <= 1e-5, turn
        w.copy_(w.flip(0))


def _shape():
    return synth.SHAPES["tiny"].with_(d=256, n_heads=4, ffn=640, vocab=1040)


def _model(sh, w, rows):
    import paper_2408_05676_amd as laser
    return laser.Model(sh.n_layers, sh.d, sh.n_heads, sh.ffn, sh.vocab, w, rows, rows, 64, eps=sh.eps, rope_base=sh.rope_base)


def _step(model, sh, rows, K=0, topk=1):
    """(accept_len, out_tokens, logits) of a step of that many rows into empty caches."""
    import paper_2408_05676_amd as laser
    B = rows // (K + 1)
    kv = gu.make_kv(sh, n_pages=4 * B, max_seqs=B, max_pages_per_seq=4)
    for s in range(B):
        kv.reserve(s, 64)
    tok = (torch.arange(B * (K + 1), device="cuda", dtype=torch.int32) * 37 % sh.vocab).view(B, K + 1)
    n = torch.full((B,), K, dtype=torch.int32, device="cuda")
    return laser.verify_step(model, kv, list(range(B)), tok[:, 0].contiguous(), tok[:, 1:].contiguous(), n, topk, -1.0, 2, want_logits=True)


@pytest.mark.parametrize("topk", [1, 2, 5])
@pytest.mark.parametrize("rows", [24, 72, 80])
def test_a_steps_head_on_the_copies(rows, topk):
    """The copies hold the values the kernels make of the caller's weights: both give the same, bit for bit."""
    sh = _shape()
    w, got = gu.gpu_weights(sh), []
    for copies in (1, 0):
        model = _model(sh, w, rows)
        model.set_option("f16_copies", copies)
        got.append(_step(model, sh, rows, 7, topk))
    assert all(torch.equal(a, b) for a, b in zip(*got))


@pytest.mark.parametrize("topk", [2, 3])
def test_long_lists_read_the_callers_head_matrix(topk):
    """A step of 17..80 rows after wlm was changed in place: with more than two entries to a list it sees the change, else the copy."""
    sh = _shape()
    w = gu.gpu_weights(sh)
    model = _model(sh, w, 24)
    new = {**w, "wlm": w["wlm"].flip(0).contiguous()}
    before, after = _step(model, sh, 24, 7, topk)[2], _step(_model(sh, new, 24), sh, 24, 7, topk)[2]
    w["wlm"].copy_(new["wlm"])
    assert torch.equal(_step(model, sh, 24, 7, topk)[2], after if topk > 2 else before) and not torch.equal(before, after)


@pytest.mark.parametrize("what", ["head 96", "step 24", "step 96"])
def test_captured_graphs_after_the_option_is_set(what):
    """A graph keeps the addresses of the copies. Setting the option leaves their memory alone; the next call makes the copies
    anew in the same place, and what is captured before that takes the caller's weights."""
    import paper_2408_05676_amd as laser
    kind, rows = what.split()[0], int(what.split()[1])
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        if kind == "head":
            w, h, drafts, n = _head(256, 1040, 12)
            h, drafts, n = h.repeat(8, 1, 1), drafts.repeat(8, 1), n.repeat(8)
            weights = {"wlm": w}
            model = laser.Model(0, 256, 4, 128, 1040, weights, rows, 8, 0)
            out = [torch.empty(8, dtype=torch.int32, device="cuda"), torch.empty((8, 12), dtype=torch.int32, device="cuda")]

            def call():
                return laser.verify_head(model, h, drafts, n, 2, -1.0, 2, want_logits=True, out=out)[2]
        else:
            sh = _shape()
            weights = gu.gpu_weights(sh)
            model = _model(sh, weights, rows)
            kv = gu.make_kv(sh, n_pages=rows, max_seqs=rows, max_pages_per_seq=1)
            for s in range(rows):
                kv.reserve(s, 16)
            tok = torch.arange(rows, device="cuda", dtype=torch.int32)
            none, n = torch.empty((rows, 0), dtype=torch.int32, device="cuda"), torch.zeros(rows, dtype=torch.int32, device="cuda")
            out = [torch.empty(rows, dtype=torch.int32, device="cuda"), torch.empty((rows, 1), dtype=torch.int32, device="cuda")]

            def call():
                return laser.verify_step(model, kv, list(range(rows)), tok, none, n, 2, -1.0, 2, want_logits=True, out=out)[2]

        def capture():
            stream.synchronize()
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=stream):
                logits = call()
            return lambda: (graph.replay(), stream.synchronize(), logits.clone())[2]

        old = call().clone()
        first = capture()
        assert torch.equal(first(), old)
        for value in (1, 0, 1):
            model.set_option("f16_copies", value)
            junk = [torch.full((t.numel(),), 7.0, dtype=torch.bfloat16, device="cuda") for t in weights.values()]   # would take freed memory
            assert torch.equal(first(), old), value
            del junk
        for t in weights.values():
            if t.dtype == torch.bfloat16:
                t.copy_(t.flip(-2))
        model.set_option("f16_copies", 1)
        second = capture()                                  # no copies: the caller's weights
        live = second()
        new = call().clone()
        assert not torch.equal(new, old) and torch.equal(first(), new)
        model.set_option("f16_copies", 0)
        assert torch.equal(call(), live) and torch.equal(second(), live) and torch.equal(first(), new)
        # (above 80 rows other tiles take the caller's weights: sums in another order)
        assert float((live.double() - new.double()).norm() / new.double().norm()) <= 1.6e-3
        stream.synchronize()


@pytest.mark.parametrize("name", ["wdown", "wlm"])
@pytest.mark.parametrize("rows", [4, 24])
def test_all_copies_or_none(name, rows):
    """One weight beyond fp16, in the last projection or in the head: up to 80 rows a step keeps no copy of any matrix."""
    import paper_2408_05676_amd as laser
    sh = synth.SHAPES["tiny"].with_(n_layers=6, d=1024, n_heads=8, ffn=4096, vocab=16384)        # copies of 200 and 32 MB
    w = gu.gpu_weights(sh)
    w[name].view(-1)[12345] = 1e5
    taken, got = [], []
    for copies in (0, 1):
        model = _model(sh, w, 96)
        model.set_option("f16_copies", copies)
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        got.append(_step(model, sh, rows)[2])
        torch.cuda.synchronize()
        taken.append(free - torch.cuda.mem_get_info()[0])
    assert torch.equal(*got) and taken[1] <= taken[0] + (8 << 20), taken
    with pytest.raises(laser.LaserError, match="fp16 range"):
        _step(model, sh, 96)


@pytest.mark.parametrize("rows", [4, 24, 96])
def test_weights_changed_in_place_without_and_with_the_option(rows):
    """Which calls see the change before the option is set, and that every route sees it afterwards."""
    import paper_2408_05676_amd as laser
    sh = _shape()
    w = gu.gpu_weights(sh)
    new = {**w, "wqkv": w["wqkv"].flip(1).contiguous(), "wlm": w["wlm"].flip(0).contiguous()}
    h = torch.ones((1, 12, sh.d), dtype=torch.float16, device="cuda")
    drafts, n = torch.zeros((1, 11), dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")

    def all_routes(model):
        got = []
        for fused in (1, 0):
            model.set_option("fused", fused)
            got.append(_step(model, sh, rows)[2])
        return got + [laser.verify_head(model, h, drafts, n, 2, -1.0, 2, want_logits=True)[2]]

    want = all_routes(_model(sh, new, max(rows, 12)))
    model = _model(sh, w, max(rows, 12))
    old = all_routes(model)
    w["wqkv"].copy_(new["wqkv"])
    w["wlm"].copy_(new["wlm"])
    kept = [True, rows > 16, False]                       # the step, the step on the general path, the head alone
    for got, before, after, copies in zip(all_routes(model), old, want, kept):
        assert torch.equal(got, before if copies else after) and not torch.equal(before, after)
    model.set_option("f16_copies", 1)
    assert all(torch.equal(got, after) for got, after in zip(all_routes(model), want))
