"""Products of 17..80 rows: the tiled kernel against the one that stages rows through registers (option mid_waves), at
the edges of its row tiles and with columns that leave a part of a tile over; and weights off the 16-byte grid, which
the tiled kernels do not take, against the same weights on it, on both sides of 80 rows."""
import pytest
import torch

import synth
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu

# Activations are rounded to fp16 (in part in two planes) at several points of a layer; another order of the sums moves
# those roundings: 2^-11 / sqrt(3) relative for a value that is rounded the other way, a small share of them in each of
# two layers. Measured between kernel choices of one step 2.4e-4 .. 4.1e-4; four times that.
TOL = 1.6e-3


def _step(model, sh, B, K, ctx=37, only=None):
    """Logits of one step of B sequences made from a fixed seed (of the sequences `only`)."""
    import paper_2408_05676_amd as laser
    kv = gu.make_kv(sh, n_pages=B * 8, max_seqs=B, max_pages_per_seq=8)
    ids = list(range(B))
    gen = torch.Generator(device="cuda").manual_seed(7)
    for s in ids:
        kv.reserve(s, 127)
    for layer in range(sh.n_layers):
        for s in ids:
            t = torch.empty((2, ctx, sh.n_heads, sh.head_dim), dtype=torch.float16, device="cuda").normal_(0.0, 1.0, generator=gen)
            kv.import_layer(s, layer, t[0], t[1])
    for s in ids:
        kv.set_len(s, ctx)
    tok = torch.randint(0, sh.vocab, (B, K + 1), generator=gen, device="cuda", dtype=torch.int32)
    n = torch.full((B,), K, dtype=torch.int32, device="cuda")
    if only is not None:
        ids, tok, n = list(only), tok[list(only)], n[list(only)]
    _, _, logits = laser.verify_step(model, kv, ids, tok[:, 0].contiguous(), tok[:, 1:].contiguous(), n, 2, 0.1, 0, want_logits=True)
    return logits.double()


def _close(x, y):
    assert torch.isfinite(x).all() and torch.isfinite(y).all()
    err = float((x - y).norm() / y.norm())
    assert err <= TOL, err


# d and ffn: reductions of 2, 4, 10 and 15 stages; 3 d and 2 ffn that are and are not multiples of 96 and 128 columns
@pytest.mark.parametrize("d,heads,ffn", [(128, 2, 128), (256, 4, 640), (640, 5, 1920), (2048, 16, 5632)])
@pytest.mark.parametrize("B,K", [(1, 16), (4, 7), (3, 10), (8, 5), (7, 6), (16, 3), (5, 12), (8, 8), (10, 7)])
def test_rows_17_to_80(d, heads, ffn, B, K):
    sh = synth.SHAPES["tiny"].with_(d=d, n_heads=heads, ffn=ffn, vocab=512)
    model = gu.make_model(sh, max_rows=80, max_batch=16, max_pos=256)
    got = _step(model, sh, B, K)
    for waves in (4, 8):
        model.set_option("mid_waves", waves)
        _close(got, _step(model, sh, B, K))


@pytest.mark.parametrize("B,K", [(4, 7), (9, 9), (13, 12)])
@pytest.mark.parametrize("copies", [0, 1])
def test_weights_off_the_16_byte_grid(B, K, copies):
    import paper_2408_05676_amd as laser
    sh = synth.SHAPES["tiny"].with_(d=256, n_heads=4, ffn=640, vocab=512)
    w = gu.gpu_weights(sh)

    def off(t):                                                 # the same values, 8 bytes further on
        flat = torch.empty(t.numel() + 4, dtype=t.dtype, device="cuda")
        flat[4:] = t.flatten()
        return flat[4:].view(t.shape)

    moved = {k: off(v) if v.dtype == torch.bfloat16 else v for k, v in w.items()}
    out = []
    for weights in (w, moved):
        model = laser.Model(sh.n_layers, sh.d, sh.n_heads, sh.ffn, sh.vocab, weights, 192, 16, 256, eps=sh.eps, rope_base=sh.rope_base)
        model.set_option("f16_copies", copies)
        out.append(_step(model, sh, B, K))
    _close(out[1], out[0])


# (entries of the tables: 17..80 rows 3; above 14 plain, 9 split, 4 head, 5, 4 and 2 of them also with bf16 weights)
def _tile_shape(**kw):
    # columns that leave a part of every tile over, reductions of four and five stages
    return synth.SHAPES["tiny"].with_(d=256, n_heads=4, ffn=640, vocab=1040, **kw)


@pytest.mark.parametrize("tile", range(1, 15))
@pytest.mark.parametrize("B,K", [(7, 12), (15, 12), (16, 25), (11, 63)])
@pytest.mark.parametrize("copies", [1, 0])
def test_every_tile_above_80_rows(tile, B, K, copies):
    """Each entry of the tile tables, with fp16 and bf16 weights, one and two planes at gate/up, one and several parts of the
    reduction: less than a tile, a tile and some, several tiles of rows; against the register-staged kernel, 78 rows at most in a call."""
    import paper_2408_05676_amd as laser
    sh = _tile_shape()
    w = gu.gpu_weights(sh)
    mk = lambda rows: laser.Model(sh.n_layers, sh.d, sh.n_heads, sh.ffn, sh.vocab, w, rows, 64, 256, eps=sh.eps, rope_base=sh.rope_base)
    few = mk(80)
    few.set_option("mid_waves", 4)
    per = max(1, 80 // (K + 1))
    want = torch.cat([_step(few, sh, B, K, only=range(b, min(b + per, B))) for b in range(0, B, per)])
    model = mk(B * (K + 1))
    model.set_option("f16_copies", copies)
    model.set_option("tile", tile)
    for split_ffn, parts in ((0, 0), (1, 1), (0, 2)):
        model.set_option("split_ffn", split_ffn)
        for name in ("ksplit_qkv", "ksplit_o", "ksplit_down"):
            model.set_option(name, parts)
        _close(_step(model, sh, B, K), want)


@pytest.mark.parametrize("tile", [1, 2, 3])
@pytest.mark.parametrize("B,K", [(1, 16), (4, 7), (3, 10), (4, 11), (7, 8), (5, 12), (8, 8), (10, 7)])
@pytest.mark.parametrize("copies", [1, 0])
def test_every_tile_of_17_to_80_rows(tile, B, K, copies):
    """With weights from the fp16 copies and from the caller's own."""
    sh = _tile_shape()
    model = gu.make_model(sh, max_rows=80, max_batch=16, max_pos=256)
    model.set_option("f16_copies", copies)
    model.set_option("tile", tile)
    got = _step(model, sh, B, K)
    model.set_option("mid_waves", 4)
    _close(got, _step(model, sh, B, K))


@pytest.mark.parametrize("tile", [1, 2, 3, 4])
@pytest.mark.parametrize("topk", [2, 5])
@pytest.mark.parametrize("copies", [1, 0])
@pytest.mark.parametrize("B,K", [(9, 8), (16, 12), (12, 40)])
def test_every_tile_of_the_head(tile, topk, copies, B, K):
    """Logits against a float64 product, and the acceptance against the rule on those logits."""
    import paper_2408_05676_amd as laser
    d, V = 256, 1040
    gen = torch.Generator(device="cuda").manual_seed(B + tile)
    w = torch.empty((V, d), dtype=torch.bfloat16, device="cuda").normal_(0.0, 0.1, generator=gen)
    h = torch.empty((B, K + 1, d), dtype=torch.float16, device="cuda").normal_(generator=gen)
    want = h.double().flatten(0, 1) @ w.double().t()
    drafts = want.view(B, K + 1, V)[:, :K].topk(topk, dim=-1).indices[..., -1].to(torch.int32)      # rank topk - 1: just inside
    drafts[:, K // 2] = want.view(B, K + 1, V)[:, K // 2].topk(topk + 1, dim=-1).indices[:, topk].to(torch.int32)   # just outside
    n = torch.full((B,), K, dtype=torch.int32, device="cuda")
    model = laser.Model(0, d, 2, 128, V, {"wlm": w}, B * (K + 1), B, 0)
    model.set_option("f16_copies", copies)
    model.set_option("tile", tile)
    acc, out, logits = laser.verify_head(model, h, drafts, n, topk, -1.0, 2, want_logits=True)
    # products of fp16 and bf16 are exact in float32, 256 of them are added in float32
    assert float((logits.double().flatten(0, 1) - want).norm() / want.norm()) <= 1e-5
    assert (acc == K // 2).all()
    assert torch.equal(out[:, :K // 2], drafts[:, :K // 2])
    assert torch.equal(out[:, K // 2], want.view(B, K + 1, V)[:, K // 2].argmax(-1).to(torch.int32))


@pytest.mark.parametrize("d,heads,ffn", [(128, 2, 128), (640, 5, 1920)])
@pytest.mark.parametrize("B,K", [(1, 0), (1, 8), (3, 4), (2, 7), (1, 16), (4, 7), (6, 7), (10, 7)])
def test_copies_up_to_80_rows(d, heads, ffn, B, K):
    """The fp16 copies hold the values that the kernels make of the bf16 weights: the same products, bit for bit (up to 16 rows
    on the persistent kernel)."""
    sh = synth.SHAPES["tiny"].with_(d=d, n_heads=heads, ffn=ffn, vocab=512)
    out = []
    for copies in (1, 0):
        model = gu.make_model(sh, max_rows=80, max_batch=16, max_pos=256)
        model.set_option("f16_copies", copies)
        out.append(_step(model, sh, B, K))
    assert torch.equal(out[0], out[1])


def test_a_weight_beyond_fp16_takes_no_copies():
    """Up to 80 rows the step does without copies; with more it is refused, as it says."""
    import paper_2408_05676_amd as laser
    sh = _tile_shape()
    w = dict(gu.gpu_weights(sh))
    w["wdown"] = w["wdown"].clone()
    w["wdown"][1, 3, 5] = 1e5
    out = []
    for copies in (1, 0):
        model = laser.Model(sh.n_layers, sh.d, sh.n_heads, sh.ffn, sh.vocab, w, 96, 16, 256, eps=sh.eps, rope_base=sh.rope_base)
        model.set_option("f16_copies", copies)
        out.append(_step(model, sh, 4, 7))
    assert torch.equal(out[0], out[1])
    model.set_option("f16_copies", 1)
    with pytest.raises(laser.LaserError, match="fp16 range"):
        _step(model, sh, 12, 7)


def _head_case(d, V, B, K, topk, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    w = torch.empty((V, d), dtype=torch.bfloat16, device="cuda").normal_(0.0, 0.1, generator=gen)
    h = torch.empty((B, K + 1, d), dtype=torch.float16, device="cuda").normal_(generator=gen)
    return w, h


@pytest.mark.parametrize("topk", [1, 2, 5])
@pytest.mark.parametrize("copies", [1, 0])
@pytest.mark.parametrize("B,K", [(1, 16), (4, 7), (3, 10), (6, 7), (9, 7), (8, 9)])
def test_head_of_17_to_80_rows(B, K, topk, copies):
    """Logits against a float64 product; drafts of rank topk - 1 pass, the one of rank topk does not. (The head alone reads the caller's
    matrix here whatever the option says; a step's head on the copies: test_gpu_weight_copies.py.)"""
    import paper_2408_05676_amd as laser
    d, V = 256, 1040
    w, h = _head_case(d, V, B, K, topk, B)
    want = h.double().flatten(0, 1) @ w.double().t()
    by_rank = want.view(B, K + 1, V)[:, :K].topk(topk + 1, dim=-1).indices.to(torch.int32)
    drafts = by_rank[..., topk - 1].contiguous()
    drafts[:, K // 2] = by_rank[:, K // 2, topk]
    n = torch.full((B,), K, dtype=torch.int32, device="cuda")
    model = laser.Model(0, d, 2, 128, V, {"wlm": w}, B * (K + 1), B, 0)
    model.set_option("f16_copies", copies)
    acc, out, logits = laser.verify_head(model, h, drafts, n, topk, -1.0, 2, want_logits=True)
    # products of fp16 and bf16 are exact in float32, 256 of them are added in float32
    assert float((logits.double().flatten(0, 1) - want).norm() / want.norm()) <= 1e-5
    assert (acc == K // 2).all()
    assert torch.equal(out[:, K // 2], want.view(B, K + 1, V)[:, K // 2].argmax(-1).to(torch.int32))


@pytest.mark.parametrize("topk", [2, 3, 8])
@pytest.mark.parametrize("B,K", [(1, 16), (8, 8), (8, 9)])
def test_long_lists_of_17_to_80_rows(B, K, topk):
    """Lists of more than two entries take the kernel that keeps them per workgroup (seen by the order of its sums: the logits are
    those of option mid_waves bit for bit), shorter ones the tiled kernel."""
    import paper_2408_05676_amd as laser
    d, V = 2048, 4112
    w, h = _head_case(d, V, B, K, topk, B)
    drafts, n = torch.zeros((B, K), dtype=torch.int32, device="cuda"), torch.full((B,), K, dtype=torch.int32, device="cuda")
    model = laser.Model(0, d, 16, 128, V, {"wlm": w}, B * (K + 1), B, 0)
    got = laser.verify_head(model, h, drafts, n, topk, -1.0, 2, want_logits=True)[2]
    model.set_option("mid_waves", 4)
    assert torch.equal(got, laser.verify_head(model, h, drafts, n, topk, -1.0, 2, want_logits=True)[2]) == (topk > 2)


@pytest.mark.parametrize("B,K", [(8, 8), (9, 10), (30, 12)])
@pytest.mark.parametrize("topk", [1, 2, 3])
def test_head_ties(B, K, topk):
    """Every logit stands twice in a lane, twice in a chunk and in another chunk: the smaller id is ahead. A row of zeros ties all."""
    import paper_2408_05676_amd as laser
    d, V = 256, 1024
    w, h = _head_case(d, V, B, K, topk, 3)
    w = w[:128].repeat_interleave(2, 0).repeat(4, 1).contiguous()                # ids 2 i, 2 i + 1, and the same 256 further on
    h[:, K] = 0                                                                  # (the last row is only read for its arg-max)
    top = (h[:, :K].double() @ w[:256:2].double().t()).argmax(-1) * 2
    order = torch.stack([top, top + 1, top + 256, top + 257], -1).to(torch.int32)
    n = torch.full((B,), K, dtype=torch.int32, device="cuda")
    model = laser.Model(0, d, 2, 128, V, {"wlm": w}, B * (K + 1), B, 0)
    acc, out = laser.verify_head(model, h, order[..., topk - 1].contiguous(), n, topk, -1.0, 2)[:2]
    assert (acc == K).all() and (out[:, K] == 0).all()
    acc, out = laser.verify_head(model, h, order[..., topk].contiguous(), n, topk, -1.0, 2)[:2]
    assert (acc == 0).all() and torch.equal(out[:, 0], order[:, 0, 0])


@pytest.mark.parametrize("topk", [1, 2, 5])
def test_head_infinities(topk):
    """Infinite and undefined logits: as the kernel for operands off the grid, whose epilogue is another one, takes them."""
    import paper_2408_05676_amd as laser
    d, V, B, K = 256, 1040, 9, 10
    w, h = _head_case(d, V, B, K, topk, 5)
    h[1, 0, 3] = float("inf")
    h[2, 0] = float("nan")
    h[3, 0, 5], h[3, 0, 6] = float("inf"), float("-inf")
    w[:, 7] = -0.25
    h[4, 0, 7] = float("inf")                                                   # every logit is -inf
    h[5, 1] = 0
    flat = torch.empty(w.numel() + 8, dtype=w.dtype, device="cuda")
    flat[1:1 + w.numel()] = w.flatten()
    drafts = torch.randint(0, V, (B, K), device="cuda", dtype=torch.int32)
    drafts[:, 0] = torch.arange(B, device="cuda", dtype=torch.int32)
    n = torch.full((B,), K, dtype=torch.int32, device="cuda")
    got = []
    for wlm, copies in ((w, 1), (flat[1:1 + w.numel()].view(w.shape), 0)):
        model = laser.Model(0, d, 2, 128, V, {"wlm": wlm}, B * (K + 1), B, 0)
        model.set_option("f16_copies", copies)
        got.append(laser.verify_head(model, h, drafts, n, topk, 0.01, 2, want_logits=True))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
    assert torch.allclose(got[0][2], got[1][2], rtol=1e-4, atol=1e-4, equal_nan=True)
