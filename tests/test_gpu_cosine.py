"""Row maxima of the sentences' Gram matrix at the edges of its tiles: numbers of sentences around 16 and 32 columns and the
128 rows of a workgroup, against fp64."""
import numpy as np
import pytest
import torch

from test_gpu_edges import _structure
from test_gpu_two_pass import _cfg, _score

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("counts", [[1, 2, 15, 16, 17], [31, 32, 33, 63, 64, 65], [127, 128, 129, 159, 160, 161, 300]])
def test_counts_of_sentences_around_the_tiles(counts):
    L, H, group, alpha = 2, 2, 4, 8
    rng = np.random.default_rng(sum(counts))
    offsets = [[0] + [int(x) for x in np.cumsum(rng.integers(1, 4, n))] for n in counts]
    offsets = [o[:-1] + [max(o[-1], alpha + n)] for o, n in zip(offsets, counts)]
    st = _structure(offsets)
    cfg = _cfg("gram", len(counts), L, H, group, alpha)
    g = torch.Generator(device="cuda")
    g.manual_seed(len(counts))
    k = torch.randn((L, H, st.total_tokens, 128), generator=g, device="cuda").to(torch.bfloat16)
    q = torch.randn((L, len(counts), H * group, alpha, 128), generator=g, device="cuda").to(torch.bfloat16)
    lam = _score(cfg, st, k, q)[1].double().cpu()
    kd = k.double().cpu()
    for b, (o, n) in enumerate(zip(offsets, counts)):
        t0, s0 = int(st.seq_off[b]), st.sent_base(b)
        for l in range(L):
            for h in range(H):
                e = torch.stack([kd[l, h, t0 + x:t0 + y].mean(0) for x, y in zip(o[:-1], o[1:])])
                e = e / e.norm(dim=1, keepdim=True)
                want = torch.where(torch.triu(torch.ones(n, n), 1) > 0, e @ e.T, torch.tensor(-np.inf, dtype=torch.float64)).max(1).values
                # unit components carry 16 bits: a cosine is within 2 * 2^-16 of the exact one (typically 1e-6)
                np.testing.assert_allclose(lam[l, h, s0:s0 + n - 1].numpy(), want[:-1].numpy(), rtol=0, atol=3.1e-5)
                assert lam[l, h, s0 + n - 1] == -np.inf
