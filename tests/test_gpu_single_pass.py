"""The single-pass scan where its work per span changes form: few and many sentences in a span (4, 8 or 16 lanes per
sentence mean, one to four registers of key sums), spans of one to eight stages whose loads run on into the next item, last
stages of every length, group sizes with rows of padding, and more items than workgroups."""
import numpy as np
import pytest
import torch

from paper_2512_07993_amd import binding as B
from paper_2512_07993_amd import workloads as W

from helpers import compare_head, oracle_head, run_step
from test_gpu_edges import _random_kvq, _structure

pytestmark = pytest.mark.gpu


def _offsets(rng):
    """Sequences whose spans hold 1, 2, 4, 5, 8, 9 and 16 sentences, and one of all sorts."""
    seqs = []
    for length in (128, 64, 32, 25, 16, 14, 8, 3, 1):
        n = int(rng.integers(40, 700))
        seqs.append(sorted(set(range(0, n, length)) | {n}))
    off = [0]
    while off[-1] < 2300:
        off.append(off[-1] + int(rng.choice([1, 2, 7, 15, 16, 17, 33, 64, 100, 127, 128])))
    seqs.append(off)
    return seqs


@pytest.mark.parametrize("dtype,group,alpha", [("bf16", 4, 16), ("bf16", 7, 8), ("bf16", 3, 13), ("bf16", 1, 3), ("bf16", 8, 7), ("f32", 4, 8)])
def test_spans_of_every_shape(dtype, group, alpha):
    rng = np.random.default_rng(group * 100 + alpha)
    st = _structure(_offsets(rng))
    layers = 24  # 24 x 2 heads of about 14 items each
    cfg = W.Config("spans", 7, len(st.seq_len), layers, 2, 2 * group, dtype, 0, 0, 150, alpha, 40, 20.0, 0.0)
    k0, v0, q = _random_kvq(cfg, st, 5)
    k, v = k0.clone(), v0.clone()
    out = run_step(cfg, st, k, v, q)
    assert int(out.dev_status.item()) == 0
    stats = {}
    for l in (0, 11, layers - 1):
        for b in range(cfg.batch):
            compare_head(cfg, st, out, k, v, k0, v0, oracle_head(cfg, st, k0, v0, q, l, l % 2, b), l, l % 2, b, stats)
    # the rest of the heads: the two-pass scan, which forms the same quantities in another order (fp32 sums: 1e-5)
    k2, v2 = k0.clone(), v0.clone()
    two = run_step(cfg, st, k2, v2, q, flags=B.FLAG_FORCE_TWO_PASS)
    assert torch.allclose(out.tok_imp, two.tok_imp, rtol=1e-5, atol=1e-9)
    lam = torch.isfinite(two.sent_lambda)
    assert torch.equal(torch.isfinite(out.sent_lambda), lam)
    assert torch.allclose(out.sent_lambda[lam], two.sent_lambda[lam], rtol=0, atol=1e-5)
