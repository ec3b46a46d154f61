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


def _step(model, sh, B, K, ctx=37):
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
