"""The two-pass scan of bf16 caches where its statistics can go wrong: runs of several chunks, rows that see none of
a chunk, sums near the end of the fp32 range, rows of very different scale, large and infinite keys."""
import numpy as np
import pytest
import torch

import oracle
from paper_2512_07993_amd import binding as B
from paper_2512_07993_amd import workloads as W
from helpers import make_cache
from test_gpu_edges import _structure

pytestmark = pytest.mark.gpu
TWO = B.FLAG_FORCE_TWO_PASS


def _score(cfg, st, k, q, flags=0, ranges=None):
    """Scores, lambdas, token importance (V is not read)."""
    cache = make_cache(cfg, st, k, k)
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    params = B.Params(cfg.obs_window, cfg.protect_window, max(cfg.budget, cfg.protect_window), dev_status=status, flags=flags)
    out = [torch.full((cfg.n_layers, cfg.n_kv_heads, n), float("nan"), dtype=torch.float32, device="cuda")
           for n in (st.total_sentences, st.total_sentences, st.total_tokens)]
    if ranges is None:
        ws = torch.empty(B.skipkv_workspace_bytes(cache, params), dtype=torch.uint8, device="cuda")
        B.skipkv_score(cache, params, q, None, *out, ws)
    else:
        ws = torch.empty(B.skipkv_ranges_workspace_bytes(cache, params), dtype=torch.uint8, device="cuda")
        B.skipkv_score_ranges(cache, ranges, params, q, None, *out, ws)
    torch.cuda.synchronize()
    assert int(status.item()) == 0
    return out


def _cfg(name, batch, L, H, group, alpha, protect=40):
    return W.Config(name, 9, batch, L, H, H * group, "bf16", 0, 0, 96, alpha, max(alpha, protect), 16.0, 0.0)


def _long_batch(L, H):
    """Sequences of ragged lengths, in such numbers that runs of several chunks pay."""
    rng = np.random.default_rng(3)
    offsets = []
    for n in [9500, 1500, 700, 8100, 260, 5333, 9001, 40, 7000, 3100, 6600, 9100, 4700, 2900]:
        off = [0]
        while off[-1] < n:
            off.append(min(n, off[-1] + int(rng.integers(1, 50))))
        offsets.append(off)
    st = _structure(offsets)
    assert L * H * (st.total_tokens // 256) >= 2 * 8 * 512
    return offsets, st


def _bits(t):
    return t.view(torch.int32)


@pytest.mark.parametrize("group,alpha", [(5, 32), (4, 16)])
def test_runs_of_chunks_give_the_same_bits_wherever_a_sequence_stands(group, alpha):
    # The plan's blocks draw their ranges of chunks in the order in which they arrive, and another order of the batch is
    # another order of the ranges: a sequence's statistics must not depend on where its chunks stand.
    L, H = 4, 8
    offsets, st = _long_batch(L, H)
    n = len(offsets)
    cfg = _cfg("runs", n, L, H, group, alpha)
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    k = torch.randn((L, H, st.total_tokens, 128), generator=g, device="cuda").to(torch.bfloat16)
    q = torch.randn((L, n, H * group, alpha, 128), generator=g, device="cuda").to(torch.bfloat16)
    ref = _score(cfg, st, k, q, TWO)
    for _ in range(3):
        for x, y in zip(ref, _score(cfg, st, k, q, TWO)):
            assert torch.equal(_bits(x), _bits(y))
    order = list(np.random.default_rng(5).permutation(n))
    st2 = _structure([offsets[b] for b in order])
    k2 = torch.cat([k[:, :, st.seq_off[b]:st.seq_off[b + 1]] for b in order], 2)
    got = _score(cfg, st2, k2, q[:, order].contiguous(), TWO)
    for j, b in enumerate(order):
        for x, y, per_tok in zip(ref, got, (False, False, True)):
            a, c = (int(st.seq_off[b]), int(st2.seq_off[j])) if per_tok else (st.sent_base(b), st2.sent_base(j))
            m = int(st.seq_len[b]) if per_tok else int(st.n_sent[b])
            assert torch.equal(_bits(x[..., a:a + m]), _bits(y[..., c:c + m])), (b, j, per_tok)
    # every head a sequence of its own
    ranges = B.Ranges(*[torch.from_numpy(x.astype(np.int32)).cuda().expand(L, H, x.size).contiguous() for x in (st.seq_len, st.n_sent, st.sent_off)])
    for _ in range(2):
        for x, y in zip(ref, _score(cfg, st, k, q, TWO, ranges)):
            assert torch.equal(_bits(x), _bits(y))


def test_jumping_logits_in_runs_of_several_chunks():
    # half of the queries see logits 200 log2 units above the first ones from some token of a run on, the other half as
    # far below: the run's sums are done again with references that follow the logits
    L, H, group, alpha = 4, 8, 5, 32
    offsets, st = _long_batch(L, H)
    n = len(offsets)
    cfg = _cfg("run-jumps", n, L, H, group, alpha)
    g = torch.Generator(device="cuda")
    g.manual_seed(2)
    k = torch.randn((L, H, st.total_tokens, 128), generator=g, device="cuda").to(torch.bfloat16)
    for b, t in ((0, 300), (0, 700), (3, 1000), (5, 17), (8, 5000)):
        k[:, :, int(st.seq_off[b]) + t, 0] = 40.0
    q = torch.randn((L, n, H * group, alpha, 128), generator=g, device="cuda").to(torch.bfloat16)
    q[..., 0::2, :, 0] = 40.0
    q[..., 1::2, :, 0] = -40.0
    imp = _score(cfg, st, k, q, TWO)[2]
    for l, h, b in ((0, 0, 0), (3, 7, 0), (1, 2, 3), (2, 5, 5), (0, 1, 8), (3, 3, 1)):
        t0, t1 = int(st.seq_off[b]), int(st.seq_off[b + 1])
        want = oracle.token_importance(q[l, b, h * group:(h + 1) * group].double().cpu().numpy(), k[l, h, t0:t1].double().cpu().numpy())
        np.testing.assert_allclose(imp[l, h, t0:t1].cpu().numpy(), want, rtol=1e-3, atol=1e-12)


@pytest.mark.parametrize("block_size", [16, 24])
@pytest.mark.parametrize("group,alpha", [(5, 32), (4, 16)])
def test_jumping_logits_on_pages(group, alpha, block_size):
    from test_gpu_paged import _run_paged, _to_pages
    st = _structure([[0, 600, 610, 680, 777], [0, 5, 700, 1000], [0, 17]])  # (sentences that the single-pass scan leaves)
    cfg = _cfg("page-jumps", 3, 1, 2, group, alpha)
    g = torch.Generator(device="cuda")
    g.manual_seed(8)
    k = torch.randn((1, 2, st.total_tokens, 128), generator=g, device="cuda").to(torch.bfloat16)
    k[:, :, [40, 650, 800, 1500], 0] = 40.0
    q = torch.randn((1, 3, 2 * group, alpha, 128), generator=g, device="cuda").to(torch.bfloat16)
    q[..., 0] = 40.0
    kp, vp, table = _to_pages(cfg, st, k, k, block_size, seed=4)
    imp = _run_paged(cfg, st, kp, vp, table, q).tok_imp
    for h in range(2):
        for b in range(3):
            t0, t1 = int(st.seq_off[b]), int(st.seq_off[b + 1])
            want = oracle.token_importance(q[0, b, h * group:(h + 1) * group].double().cpu().numpy(), k[0, h, t0:t1].double().cpu().numpy())
            np.testing.assert_allclose(imp[0, h, t0:t1].cpu().numpy(), want, rtol=1e-3, atol=1e-12)


def test_a_row_that_sees_none_of_a_chunk_keeps_its_own_reference():
    # The last chunk begins inside the observation window: its first window queries see none of it, the others see logits
    # 250 log2 units above everything before.
    group, alpha = 5, 32
    st = _structure([[0, 128, 256, 384, 512, 538]])
    cfg = _cfg("hidden", 1, 1, 1, group, alpha)
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    k = torch.randn((1, 1, 538, 128), generator=g, device="cuda").to(torch.bfloat16)
    q = torch.randn((1, 1, group, alpha, 128), generator=g, device="cuda").to(torch.bfloat16)
    k[..., :512, 0] = 0.0
    k[..., 512:, 0] = 50.0
    q[..., 0] = 40.0
    imp = _score(cfg, st, k, q)[2]
    want = oracle.token_importance(q[0, 0].double().cpu().numpy(), k[0, 0].double().cpu().numpy())
    np.testing.assert_allclose(imp[0, 0].cpu().numpy(), want, rtol=1e-3, atol=1e-12)


@pytest.mark.parametrize("flags", [0, TWO])
@pytest.mark.parametrize("group,alpha", [(5, 32), (4, 16), (4, 32), (7, 8)])
def test_sums_near_the_end_of_the_range_can_still_be_added(group, alpha, flags):
    # All logits are 0 but those of two tokens, at 127.5 log2 units: either term fits fp32, their sum does not.  The
    # tokens are in one span or chunk, in shares of different waves of a tile, or in different spans and chunks.
    st = _structure([[0, 64, 128, 192, 256, 320, 400, 500]])
    cfg = _cfg("range", 1, 1, 1, group, alpha)
    for where in ((70, 100), (70, 120), (80, 96), (70, 130), (70, 300)):
        k = torch.zeros((1, 1, 500, 128), dtype=torch.bfloat16, device="cuda")
        q = torch.zeros((1, 1, group, alpha, 128), dtype=torch.bfloat16, device="cuda")
        q[..., 0] = 40.0
        k[..., list(where), 0] = 25.0
        imp = _score(cfg, st, k, q, flags)[2]
        want = oracle.token_importance(q[0, 0].double().cpu().numpy(), k[0, 0].double().cpu().numpy())
        np.testing.assert_allclose(imp[0, 0].cpu().numpy(), want, rtol=1e-3, atol=1e-12)


@pytest.mark.parametrize("group,alpha", [(5, 32), (8, 32)])
def test_normalisers_of_rows_next_to_rows_of_another_scale(group, alpha):
    # One head of the group has logits 20 times as large as the others.  Where the others decide the maximum over the
    # group, the importance carries the error of their normalisers, the same for all tokens of a query.  A normaliser and
    # its difference to a logit lie between 8 and 16 log2 units: half a unit in the last place of fp32 there is 4.8e-7, two
    # of them are a relative error of 2 x 4.8e-7 x ln 2 = 6.6e-7.
    N = 4000
    st = _structure([list(range(0, N + 1, 20))])
    cfg = _cfg("scales", 1, 1, 4, group, alpha)
    g = torch.Generator(device="cuda")
    g.manual_seed(4)
    k = torch.randn((1, 4, N, 128), generator=g, device="cuda").to(torch.bfloat16)
    q = torch.randn((1, 1, 4 * group, alpha, 128), generator=g, device="cuda").to(torch.bfloat16)
    q[:, :, 0::group] *= 20.0
    imp = _score(cfg, st, k, q, TWO)[2]
    err = []
    for h in range(4):
        want = oracle.token_importance(q[0, 0, h * group:(h + 1) * group].double().cpu().numpy(), k[0, h].double().cpu().numpy())
        rel = imp[0, h].double().cpu().numpy() / want - 1.0
        err.append(abs(np.median(rel)))
    assert max(err) < 7e-7


def test_embeddings_of_large_keys():
    # the mean of a sentence of 400 keys of 1e17 has a square that fits, their sum has not
    st = _structure([[0, 400, 420, 820, 900]])
    cfg = _cfg("large", 1, 1, 1, 4, 16)
    g = torch.Generator(device="cuda")
    g.manual_seed(6)
    base = torch.randn(128, generator=g, device="cuda")
    k = ((base + 0.5 * torch.randn((1, 1, 900, 128), generator=g, device="cuda")) * 1e17).to(torch.bfloat16)
    q = (torch.randn((1, 1, 4, 16, 128), generator=g, device="cuda") * 1e-17).to(torch.bfloat16)
    lam = _score(cfg, st, k, q, TWO)[1][0, 0].cpu().numpy()
    want = oracle.sentence_redundancy(oracle.sentence_embeddings(k[0, 0].double().cpu().numpy(), st.offsets(0).astype(np.int64)))
    np.testing.assert_allclose(lam[:-1], want[:-1], rtol=1e-3, atol=1e-5)


@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("group,alpha", [(4, 16), (5, 32)])
@pytest.mark.parametrize("token", [305, 560, 899, 640])
def test_an_infinite_key_stays_in_its_sentence(group, alpha, token, paged):
    # A key with an infinity that every query scores -inf has weight 0 and spoils the embedding of its own sentence only.
    # (One of the chunks has more than 16 sentences, which other waves sum.)
    off = [0, 300, 310, 330, 335] + list(range(350, 621, 9)) + [640, 660, 700, 900, 930, 1000]
    st = _structure([off])
    cfg = _cfg("inf", 1, 1, 1, group, alpha)
    g = torch.Generator(device="cuda")
    g.manual_seed(7)
    k = torch.randn((1, 1, 1000, 128), generator=g, device="cuda").to(torch.bfloat16)
    q = torch.randn((1, 1, group, alpha, 128), generator=g, device="cuda").to(torch.bfloat16)
    q[..., 5] = 1.0
    k[0, 0, token, 5] = float("-inf")
    if paged:
        from test_gpu_paged import _run_paged, _to_pages
        kp, vp, table = _to_pages(cfg, st, k, k, 24, seed=3)
        out = _run_paged(cfg, st, kp, vp, table, q)
        lam, imp = out.sent_lambda, out.tok_imp
    else:
        _, lam, imp = _score(cfg, st, k, q, TWO)
    lam, imp = lam[0, 0].cpu().numpy(), imp[0, 0].cpu().numpy()
    x = k[0, 0].double().cpu().numpy()
    x[token, 5] = -1e30
    np.testing.assert_allclose(imp, oracle.token_importance(q[0, 0].double().cpu().numpy(), x), rtol=1e-3, atol=1e-12)
    bad = int(np.searchsorted(off, token, side="right")) - 1
    emb = oracle.sentence_embeddings(x, np.asarray(off))
    good = [s for s in range(len(off) - 1) if s != bad]
    want = oracle.sentence_redundancy(emb[good])
    np.testing.assert_allclose(lam[good][:-1], want[:-1], rtol=1e-3, atol=1e-5)


@pytest.mark.parametrize("group,alpha", [(5, 32), (4, 8)])
def test_sentences_that_begin_and_end_anywhere_in_a_tile(group, alpha):
    # Lengths 1, 2, ... put first and last tokens at every place of the 16-token stages and the 64-token tiles; one
    # sentence is longer than a chunk, so that it holds whole tiles and its bounds lie far outside of others.
    L, H = 1, 2
    lengths = list(range(1, 40)) + [700] + list(range(40, 1, -3)) + [64, 16, 128, 1]
    offsets = [list(np.cumsum([0] + lengths)), list(np.cumsum([0, 15, 1, 16, 32, 64, 3]))]
    st = _structure([[int(x) for x in o] for o in offsets])
    cfg = _cfg("bounds", 2, L, H, group, alpha)
    g = torch.Generator(device="cuda")
    g.manual_seed(4)
    k = torch.randn((L, H, st.total_tokens, 128), generator=g, device="cuda").to(torch.bfloat16)
    q = torch.randn((L, 2, H * group, alpha, 128), generator=g, device="cuda").to(torch.bfloat16)
    lam = _score(cfg, st, k, q, TWO)[1].double().cpu()
    kd = k.double().cpu()
    for b, o in enumerate(offsets):
        t0, s0, n = int(st.seq_off[b]), st.sent_base(b), int(st.n_sent[b])
        for h in range(H):
            e = torch.stack([kd[0, h, t0 + x:t0 + y].mean(0) for x, y in zip(o[:-1], o[1:])])
            e = e / e.norm(dim=1, keepdim=True)
            want = torch.where(torch.triu(torch.ones(n, n), 1) > 0, e @ e.T, torch.tensor(-np.inf, dtype=torch.float64)).max(1).values
            # unit components carry 16 bits: a cosine is within 2 * 2^-16 of the exact one (typically 1e-6); a token too many or
            # too few moves an embedding of n tokens by 1 / sqrt(n) > 0.03
            np.testing.assert_allclose(lam[0, h, s0:s0 + n - 1].numpy(), want[:-1].numpy(), rtol=0, atol=3.1e-5)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("L,H", [(1, 1), (1, 3), (8, 8), (43, 6), (96, 8)])  # the last one: 4096 workgroups instead of 1024
def test_sequences_that_the_single_pass_scan_leaves_get_what_the_two_pass_scan_alone_gives(dtype, L, H):
    # A head's runs (fp32: chunks) are taken from another one on than the head's before: each of them once, whatever their number
    # and that of the workgroups.  Here two to five of eight sequences are left, for a sentence that no item holds.
    rng = np.random.default_rng(L + H)
    offsets = []
    for i, n in enumerate([900, 2048, 300, 1500, 700, 2600, 40, 1025]):
        off = [0] if i % 2 and n < 1026 + 500 * (L % 3) else [0, 600]
        while off[-1] < n:
            off.append(min(n, off[-1] + int(rng.integers(1, 50))))
        offsets.append(off)
    st = _structure(offsets)
    cfg = W.Config("left", 9, 8, L, H, 4 * H, dtype, 0, 0, 96, 8, 40, 16.0, 0.0)
    g = torch.Generator(device="cuda")
    g.manual_seed(L)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    k = torch.randn((L, H, st.total_tokens, 128), generator=g, device="cuda").to(dt)
    q = torch.randn((L, 8, 4 * H, 8, 128), generator=g, device="cuda").to(dt)
    got, two = _score(cfg, st, k, q), _score(cfg, st, k, q, TWO)
    assert not any(torch.isnan(x).any() for x in got)
    for b, off in enumerate(offsets):
        s = slice(st.sent_base(b), st.sent_base(b) + int(st.n_sent[b]))
        t = slice(int(st.seq_off[b]), int(st.seq_off[b + 1]))
        for x, y, at in zip(got, two, (s, s, t)):
            if off[1] == 600:
                assert torch.equal(_bits(x[..., at]), _bits(y[..., at]))
            else:  # fp32 sums in another order
                assert torch.allclose(x[..., at], y[..., at], rtol=1e-5, atol=1e-5)


@pytest.mark.parametrize("L,H,group,alpha,n", [(1, 1, 5, 32, 9000), (1, 3, 4, 16, 20000), (1, 2, 8, 32, 520), (3, 1, 1, 1, 250), (2, 8, 5, 32, 40000), (1, 2, 8, 32, 140000)])
def test_records_of_few_and_many_runs(L, H, group, alpha, n):
    # A head's records are merged by the threads that a row has, in shares (one run, fewer runs than shares, shares of several
    # runs), or by a kernel of its own (the last two).  The normaliser and its difference to a logit are below 32 log2 units: one unit
    # in the last place of fp32 there is 1.9e-6, two of them a relative error of 2.6e-6, which all tokens of a row share; the sums of n
    # terms and products of 128 add some 1e-6 each.
    st = _structure([list(range(0, n, 50)) + [n], [0, 600, 700]])
    cfg = _cfg("records", 2, L, H, group, alpha)
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    k = torch.randn((L, H, st.total_tokens, 128), generator=g, device="cuda").to(torch.bfloat16)
    k[:, :, n // 3] *= 4.0  # (a reference of one run that the others' are far from)
    q = torch.randn((L, 2, H * group, alpha, 128), generator=g, device="cuda").to(torch.bfloat16)
    imp = _score(cfg, st, k, q, TWO)[2]
    for b in range(2):
        t0, t1 = int(st.seq_off[b]), int(st.seq_off[b + 1])
        x = torch.einsum("qd,td->qt", q[-1, b, (H - 1) * group:].reshape(group * alpha, 128).double(), k[-1, -1, t0:t1].double()) / 128 ** 0.5
        x = x.view(group, alpha, t1 - t0)
        seen = torch.arange(t1 - t0, device="cuda")[None, :] <= t1 - t0 - alpha + torch.arange(alpha, device="cuda")[:, None]
        want = torch.where(seen, x, float("-inf")).softmax(-1).amax(0).mean(0)
        assert torch.allclose(imp[-1, -1, t0:t1].double(), want, rtol=1e-5, atol=1e-12)
