"""The acceptance walk, a lane per node: chains of one, 31 and the most drafts, broken at every place."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [1, 31, 63])
def test_acceptance_walk(K):
    """Hidden states along the head's rows decide which drafts pass: chains broken at every place."""
    import paper_2408_05676_amd as laser
    rng = np.random.default_rng(K)
    V, d, B = 512, 128, 65
    w = torch.randn(V, d, generator=torch.Generator().manual_seed(1)).to(torch.bfloat16).cuda()
    model = laser.Model(0, d, d // 64, 128, V, {"wlm": w}, B * (K + 1), B, 0)
    tok = rng.integers(0, V, (B, K + 1))
    h = (w[torch.from_numpy(tok).cuda()].float() * 0.5).to(torch.float16)
    best = (h.double() @ w.double().T).argmax(-1).cpu().numpy()          # what every row would emit
    drafts = best[:, :K].astype(np.int32).copy()
    brk = np.arange(B) % (K + 1)
    for b in range(B):
        if brk[b] < K:
            drafts[b, brk[b]] = (drafts[b, brk[b]] + 1) % V
    n = torch.full((B,), K, dtype=torch.int32, device="cuda")
    acc, out, *_ = laser.verify_head(model, h, torch.from_numpy(drafts).cuda(), n, 1, 0.0, 0)
    acc, out = acc.cpu().numpy(), out.cpu().numpy()
    assert (acc == brk).all()
    for b in range(B):
        a = brk[b]
        assert (out[b, :a] == drafts[b, :a]).all() and out[b, a] == best[b, a] and (out[b, a + 1:] == -1).all()
