"""Cache pages as every writer and reader of them sees them: keys and values brought in by laser_kv_import, rows written by the
step itself (persistent and general kernels, 16 rows and fewer, and more), read back by the next step; against the oracle."""
import numpy as np
import pytest
import torch

import synth
from oracle.decoder import Decoder
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


# both head sizes; committed lengths at the edges of pages and of a wave's pair of pages; new rows inside one page, over two and over three
@pytest.mark.parametrize("heads", [4, 2])
@pytest.mark.parametrize("fused", [1, 0])
@pytest.mark.parametrize("ctx,K", [(1, 3), (15, 1), (16, 15), (31, 7), (45, 19), (270, 4)])
def test_imported_and_written_pages(heads, fused, ctx, K):
    import paper_2408_05676_amd as laser
    sh = synth.SHAPES["tiny"].with_(d=256, n_heads=heads, ffn=640, vocab=512)
    model = gu.make_model(sh, max_rows=32, max_batch=1, max_pos=512)
    model.set_option("fused", fused)
    kv = gu.make_kv(sh, n_pages=24, max_seqs=1, max_pages_per_seq=24)
    kv.reserve(0, ctx + 2 * (K + 1))
    dec = Decoder(sh.n_layers, sh.d, sh.n_heads, sh.ffn, sh.vocab, synth.gen_all_weights(sh), sh.eps, sh.rope_base)
    cache = dec.new_cache(ctx + 2 * (K + 1))
    gen = torch.Generator().manual_seed(ctx)
    for layer in range(sh.n_layers):
        t = torch.randn((2, ctx, sh.n_heads, sh.head_dim), generator=gen).to(torch.float16)
        cache.k[layer, :ctx], cache.v[layer, :ctx] = t[0].double().numpy(), t[1].double().numpy()
        t = t.cuda()
        kv.import_layer(0, layer, t[0], t[1])
    cache.commit(ctx)
    kv.set_len(0, ctx)
    n = torch.full((1,), K, dtype=torch.int32, device="cuda")
    for step in range(2):                            # the second step reads the pages the first one wrote
        tok = torch.randint(0, sh.vocab, (1, K + 1), generator=gen, dtype=torch.int32)
        _, _, logits = laser.verify_step(model, kv, [0], tok[:, 0].cuda(), tok[:, 1:].contiguous().cuda(), n, 1, -1.0, 0, want_logits=True)
        laser.kv_commit(kv, [0], n)
        want = dec.verify_forward(cache, tok[0].numpy())
        cache.commit(K + 1)
        ok, err, ratio = gu.logits_close(logits.cpu().numpy().reshape(want.shape).astype(np.float64), want)
        assert ok, (step, err, ratio)


@pytest.mark.parametrize("heads", [4, 2])
@pytest.mark.parametrize("ctx,first", [(1, 1), (7, 3), (16, 5), (21, 6), (47, 33)])
def test_import_off_the_grid_and_over_a_part(heads, ctx, first):
    """Arrays aligned to their elements only give the same pages, and an import of the first tokens leaves the others as they are."""
    import paper_2408_05676_amd as laser
    sh = synth.SHAPES["tiny"].with_(d=256, n_heads=heads, ffn=640, vocab=512)
    model = gu.make_model(sh, max_rows=4, max_batch=1, max_pos=128)
    gen = torch.Generator(device="cuda").manual_seed(ctx)
    k, v = torch.empty((2, sh.n_layers, ctx, heads, sh.head_dim), dtype=torch.float16, device="cuda").normal_(generator=gen)
    tok, n = torch.full((1, 1), 7, dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
    got = []
    for off in (0, 1, 3):
        kv = gu.make_kv(sh, n_pages=4, max_seqs=1, max_pages_per_seq=4)
        kv.reserve(0, ctx + 4)
        for layer in range(sh.n_layers):
            if off == 0:
                kv.import_layer(0, layer, k[layer], v[layer])
                continue
            for count, scale in ((ctx, 1), (first, 2), (first, 1)):            # the first tokens: others over them, then the same again
                a, b = (torch.empty(off + count * 256, dtype=torch.float16, device="cuda")[off:].view(count, heads, -1) for _ in range(2))
                a.copy_(k[layer, :count] * scale)
                b.copy_(v[layer, :count] * scale)
                kv.import_layer(0, layer, a, b)
        kv.set_len(0, ctx)
        got.append(laser.verify_step(model, kv, [0], tok[:, 0].contiguous(), tok[:, :0].contiguous(), n, 1, -1.0, 0, want_logits=True)[2].clone())
    assert torch.equal(got[0], got[1]) and torch.equal(got[0], got[2])


@pytest.mark.parametrize("rows", [4, 24, 96])
def test_weights_changed_in_place_are_seen_after_the_option_is_set(rows):
    """A step before and after: the fp16 copies are made anew, and without copies the weights are the caller's own."""
    import paper_2408_05676_amd as laser
    sh = synth.SHAPES["tiny"].with_(d=256, n_heads=4, ffn=640, vocab=512)
    w, other = gu.gpu_weights(sh), gu.gpu_weights(sh.with_(vocab=512))
    other["wqkv"], other["wlm"] = other["wqkv"].flip(1).contiguous(), other["wlm"].flip(0).contiguous()
    tok = torch.arange(rows, device="cuda", dtype=torch.int32)[:, None]

    def logits(model):
        kv = gu.make_kv(sh, n_pages=rows, max_seqs=rows, max_pages_per_seq=1)
        for s in range(rows):
            kv.reserve(s, 16)
        none = torch.empty((rows, 0), dtype=torch.int32, device="cuda")
        return laser.verify_step(model, kv, list(range(rows)), tok[:, 0].contiguous(), none, torch.zeros(rows, dtype=torch.int32, device="cuda"),
                                 1, -1.0, 0, want_logits=True)[2].clone()

    def make(weights):
        return laser.Model(sh.n_layers, sh.d, sh.n_heads, sh.ffn, sh.vocab, weights, rows, rows, 64, eps=sh.eps, rope_base=sh.rope_base)

    model, want = make(w), logits(make(other))
    logits(model)
    w["wqkv"].copy_(other["wqkv"])
    w["wlm"].copy_(other["wlm"])
    model.set_option("f16_copies", 1)
    assert torch.equal(logits(model), want)
