"""Values written into cache pages by steps of many rows, at several alignments of the committed length to the pages:
one big step against the same tokens in small ones."""
import pytest
import torch

import synth
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu
TOL = 1.6e-3          # as for any two kernel choices of one step: fp16 roundings of activations that fall the other way


@pytest.mark.parametrize("B,chunk", [(1, 17), (2, 33), (3, 48), (4, 64), (2, 50)])
@pytest.mark.parametrize("first", [0, 1, 7, 15])
def test_prompts_in_big_and_small_steps(B, chunk, first):
    import paper_2408_05676_amd as laser
    sh = synth.SHAPES["tiny"]
    T = 131
    prompts = [synth.uniform_tokens(5, 60 + b, 0, T, sh.vocab) for b in range(B)]
    ids = list(range(B))
    out = []
    for c in (chunk, 5):
        model = gu.make_model(sh, max_rows=max(16, B * 64), max_batch=B, max_pos=256)
        model.set_option("fused", 0)
        kv = gu.make_kv(sh, n_pages=B * 16, max_seqs=B, max_pages_per_seq=16)
        for s in ids:
            kv.reserve(s, 200)
        if first:          # an odd number of tokens first, so that the big steps begin inside a page
            gu.prefill(model, kv, ids, [p[:first + 1] for p in prompts], chunk=first)
        pend = gu.prefill(model, kv, ids, [p[first:] for p in prompts], chunk=c)
        none = torch.empty((B, 0), dtype=torch.int32, device="cuda")
        _, _, logits = laser.verify_step(model, kv, ids, pend, none, torch.zeros(B, dtype=torch.int32, device="cuda"), 1, -1.0, 0, want_logits=True)
        out.append(logits.double())
    assert float((out[0] - out[1]).norm() / out[1].norm()) <= TOL
