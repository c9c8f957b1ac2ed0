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


def _cut_offsets():
    """Sentences of several spans: every length around a span's edge, at every place within an item, alone, side by side,
    first, last and with others too short for a stage between them."""
    seqs = []
    for n in (128, 129, 255, 256, 257, 384, 385, 511, 512):
        seqs.append([0, n])
        seqs.append([0, 40, 40 + n, 43 + n])
    seqs.append([0, 300, 600, 900, 901, 1413, 1500])
    seqs.append([0, 100, 200, 300, 812, 830])                      # three spans, then one that needs a whole item
    off, rng = [0], np.random.default_rng(8)
    while off[-1] < 6000:
        off.append(off[-1] + int(rng.choice([5, 17, 31, 60, 129, 200, 333, 400, 512], p=[.2, .2, .2, .2, .05, .05, .05, .025, .025])))
    seqs.append(off)
    seqs.append([0, 20, 533, 600])                                 # 513 tokens: the two-pass scan's
    return seqs


@pytest.mark.parametrize("dtype,group,alpha", [("bf16", 4, 16), ("bf16", 7, 8), ("bf16", 2, 5), ("f32", 4, 8)])
def test_sentences_of_several_spans(dtype, group, alpha):
    st = _structure(_cut_offsets())
    cfg = W.Config("cut", 7, len(st.seq_len), 3, 2, 2 * group, dtype, 0, 0, 700, alpha, 40, 20.0, 0.0)
    k0, v0, q = _random_kvq(cfg, st, 6)
    k, v = k0.clone(), v0.clone()
    red = torch.rand((3, 2, st.total_tokens), device="cuda")
    out = run_step(cfg, st, k, v, q, red=red)
    assert int(out.dev_status.item()) == 0
    stats = {}
    for l in range(3):
        for b in range(cfg.batch):
            compare_head(cfg, st, out, k, v, k0, v0, oracle_head(cfg, st, k0, v0, q, l, 1, b, red=red), l, 1, b, stats)


def test_more_cut_sentences_than_there_is_room_for_items_take_the_two_pass_scan():
    # one token, then 385: eight spans for 386 tokens, where there is room for six
    off = [0]
    while off[-1] < 7000:
        off += [off[-1] + 1, off[-1] + 386]
    st = _structure([off, [0, 10, 395, 400]])
    cfg = W.Config("room", 7, 2, 2, 1, 4, "bf16", 0, 0, 700, 16, 40, 20.0, 0.0)
    k0, v0, q = _random_kvq(cfg, st, 7)
    k, v = k0.clone(), v0.clone()
    out = run_step(cfg, st, k, v, q)
    for b in range(2):
        compare_head(cfg, st, out, k, v, k0, v0, oracle_head(cfg, st, k0, v0, q, 1, 0, b), 1, 0, b, {})


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("token", [5, 40, 130, 355, 390, 560])
def test_an_infinite_key_stays_in_its_sentence(dtype, token):
    import oracle
    off = [0, 9, 30, 50, 350, 360, 391, 400, 640, 700]
    st = _structure([off])
    cfg = W.Config("inf", 7, 1, 1, 1, 4, dtype, 0, 0, 700, 8, 40, 20.0, 0.0)
    k, v, q = _random_kvq(cfg, st, 8)
    q[..., 5] = 1.0
    k[0, 0, token, 5] = float("-inf")  # every query scores it -inf: weight 0
    out = run_step(cfg, st, k.clone(), v, q)
    x = k[0, 0].double().cpu().numpy()
    x[token, 5] = -1e30
    imp = oracle.token_importance(q[0, 0].double().cpu().numpy(), x)
    np.testing.assert_allclose(out.tok_imp[0, 0].cpu().numpy(), imp, rtol=1e-3, atol=1e-12)
    bad = int(np.searchsorted(off, token, side="right")) - 1
    good = [s for s in range(len(off) - 1) if s != bad]
    want = oracle.sentence_redundancy(oracle.sentence_embeddings(x, np.asarray(off))[good])
    lam = out.sent_lambda[0, 0].cpu().numpy()
    np.testing.assert_allclose(lam[good][:-1], want[:-1], rtol=1e-3, atol=1e-5)


@pytest.mark.parametrize("n_seqs", [40, 1000])
def test_fp32_items_that_would_stay_nearly_empty_are_left_to_the_two_passes_in_large_calls(n_seqs):
    # 8 heads, below and above the 400 000 keys from which on the plan looks at how full the items are: 150 and 154 tokens an item
    # are too few, 258 and what is not cut are not
    import oracle
    kinds = [[129, 21], [40, 129, 10, 129], [129, 129], [129] * 4, [60, 70, 80]]
    offsets = [[0] + [int(x) for x in np.cumsum(kinds[i % 5])] for i in range(n_seqs)]
    st = _structure(offsets)
    assert (8 * st.total_tokens > 400000) == (n_seqs == 1000)
    cfg = W.Config("empty", 7, n_seqs, 1, 8, 8, "f32", 0, 0, 700, 4, 40, 20.0, 0.0)
    k0, v0, q = _random_kvq(cfg, st, 9)
    one = run_step(cfg, st, k0.clone(), v0.clone(), q)
    two = run_step(cfg, st, k0.clone(), v0.clone(), q, flags=B.FLAG_FORCE_TWO_PASS)
    assert int(one.dev_status.item()) == 0
    same = [torch.equal(one.tok_imp[..., t0:t1], two.tok_imp[..., t0:t1]) for t0, t1 in zip(st.seq_off[:-1], st.seq_off[1:])]
    assert same == [n_seqs == 1000 and i % 5 < 2 for i in range(n_seqs)]  # (another scan shows in the last bits)
    assert torch.allclose(one.tok_imp, two.tok_imp, rtol=1e-5, atol=1e-9)  # fp32 sums in another order
    lam = torch.isfinite(one.sent_lambda)
    assert torch.equal(lam, torch.isfinite(two.sent_lambda)) and torch.allclose(one.sent_lambda[lam], two.sent_lambda[lam], rtol=0, atol=1e-5)
    for b in (0, 1, 2, 3, n_seqs - 1):
        t0, t1 = int(st.seq_off[b]), int(st.seq_off[b + 1])
        want = oracle.token_importance(q[0, b, 3:4].double().cpu().numpy(), k0[0, 3, t0:t1].double().cpu().numpy())
        np.testing.assert_allclose(one.tok_imp[0, 3, t0:t1].cpu().numpy(), want, rtol=1e-4, atol=1e-12)
