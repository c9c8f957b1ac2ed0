"""GPU parity of skipkv_token_redundancy (Sec. 4.1 "Token Redundancy Score", Eq.5) against the oracle.

Tolerance: R is a mean of N softmax probabilities whose logits are cosines in [-1, 1]; the kernel
forms the dot products exactly (bf16 products, fp32 accumulation) and uses 1-ulp exp2/log2, so
rel 1e-3 (the bar for scores) leaves two orders of magnitude of room on bf16 caches.  For fp32
caches the keys are rounded to bf16 first (stated in the header): each cosine moves by up to
~1e-3, the mean over rows averages that down; the same rel 1e-3 is checked on N(0,1) keys."""
import numpy as np
import pytest
import torch

import oracle
from paper_2512_07993_amd import binding as B
from paper_2512_07993_amd import workloads as W

from helpers import make_cache
from test_gpu_edges import _structure

pytestmark = pytest.mark.gpu


def _run(cfg, st, k):
    cache = make_cache(cfg, st, k, k)
    ws = torch.empty(B.skipkv_redundancy_workspace_bytes(cache) + 256, dtype=torch.uint8, device="cuda")
    out = torch.full((cfg.n_layers, cfg.n_kv_heads, st.total_tokens), float("nan"), dtype=torch.float32, device="cuda")
    B.skipkv_token_redundancy(cache, out, ws)
    torch.cuda.synchronize()
    return out


def _check(cfg, st, k, out, heads, rtol):
    for (l, h, b) in heads:
        t0, t1 = int(st.seq_off[b]), int(st.seq_off[b + 1])
        want = oracle.token_redundancy(k[l, h, t0:t1].to(torch.float64).cpu().numpy())
        got = out[l, h, t0:t1].cpu().numpy().astype(np.float64)
        np.testing.assert_allclose(got, want, rtol=rtol, atol=0, err_msg="head (l=%d, h=%d, b=%d, N=%d)" % (l, h, b, t1 - t0))
        if t1 > t0:
            assert abs(got.sum() - 1.0) < 1e-4


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_ragged_batch_all_heads(dtype):
    # lengths around the 256-row and 64-column tile edges, a single token, an empty sequence
    lens = [1, 0, 63, 64, 65, 255, 256, 257, 700, 1]
    offsets = [[0, n] if n else [0] for n in lens]
    st = _structure(offsets)
    cfg = W.Config("tokred", 9, len(lens), 2, 2, 8, dtype, 0, 0, 64, 8, 16, 16.0, 0.0)
    g = torch.Generator(device="cuda")
    g.manual_seed(77)
    k = torch.randn((2, 2, st.total_tokens, 128), generator=g, device="cuda").to(W.torch_dtype(cfg))
    out = _run(cfg, st, k)
    heads = [(l, h, b) for l in range(2) for h in range(2) for b in range(len(lens)) if lens[b] > 0]
    _check(cfg, st, k, out, heads, 1e-3 if dtype == "f32" else 1e-4)


def test_lengths_around_wave_rows_and_diagonal_squares():
    # a wave has 32 rows, the squares on the diagonal 64: lengths that leave waves empty, half a square, and
    # column blocks right of the workgroup's own 256 rows with 1 to 64 columns
    lens = [31, 32, 33, 95, 96, 97, 127, 129, 191, 193, 287, 289, 319, 320, 321, 511, 513, 575, 577]
    st = _structure([[0, n] for n in lens])
    cfg = W.Config("tokred-edges", 9, len(lens), 1, 1, 4, "bf16", 0, 0, 64, 8, 16, 16.0, 0.0)
    g = torch.Generator(device="cuda")
    g.manual_seed(78)
    k = torch.randn((1, 1, st.total_tokens, 128), generator=g, device="cuda").to(torch.bfloat16)
    _check(cfg, st, k, _run(cfg, st, k), [(0, 0, b) for b in range(len(lens))], 1e-4)


def test_structured_keys_duplicates_and_scaling():
    # clusters of exact duplicates with wildly different norms (cosines are scale-free), plus noise rows
    rng = np.random.default_rng(3)
    base = rng.standard_normal((5, 128))
    rows = [base[i % 5] * 2.0 ** rng.integers(-6, 7) for i in range(300)] + list(rng.standard_normal((121, 128)))
    k_np = np.stack(rows).astype(np.float32)
    st = _structure([[0, len(rows)]])
    cfg = W.Config("tokred", 9, 1, 1, 1, 4, "bf16", 0, 0, 64, 8, 16, 16.0, 0.0)
    k = torch.from_numpy(k_np).cuda().to(torch.bfloat16).reshape(1, 1, len(rows), 128).contiguous()
    out = _run(cfg, st, k)
    _check(cfg, st, k, out, [(0, 0, 0)], 1e-4)
    r = out[0, 0].cpu().numpy()
    assert r[:300].min() > r[300:].max()  # members of the duplicate clusters collect more mass than any lone key


def test_config3_shape_sampled_heads():
    cfg = W.CONFIGS[3].scaled(n_layers=1, batch=4)
    st = W.make_structure(cfg)
    k0, v0, q = W.fill_cache(cfg, st, device="cuda")
    out = _run(cfg, st, k0)
    _check(cfg, st, k0, out, [(0, 0, 0), (0, 3, 1), (0, 5, 2), (0, 7, 3)], 1e-4)


def test_repeats_bit_for_bit_and_clears_its_own_workspace():
    """Only the blocks at and right of the diagonal are computed and every block adds to the totals of
    its rows AND of its columns, from many workgroups at once: the totals are 64-bit fixed-point integers,
    so the result must not depend on the order of arrival.  Two calls on the same workspace (the second
    one finds the first one's totals and factors in it), and one on a fresh, garbage-filled workspace."""
    cfg = W.CONFIGS[3].scaled(n_layers=2, batch=4)
    st = W.make_structure(cfg)
    k0, v0, q = W.fill_cache(cfg, st, device="cuda")
    cache = make_cache(cfg, st, k0, k0)
    n = B.skipkv_redundancy_workspace_bytes(cache) + 256
    ws = torch.empty(n, dtype=torch.uint8, device="cuda")
    outs = []
    for w in (ws, ws, torch.full((n,), 0xA5, dtype=torch.uint8, device="cuda")):
        out = torch.full((cfg.n_layers, cfg.n_kv_heads, st.total_tokens), float("nan"), dtype=torch.float32, device="cuda")
        B.skipkv_token_redundancy(cache, out, w)
        torch.cuda.synchronize()
        outs.append(out)
    assert not bool(torch.isnan(outs[0]).any())
    assert torch.equal(outs[0].view(torch.int32), outs[1].view(torch.int32))
    assert torch.equal(outs[0].view(torch.int32), outs[2].view(torch.int32))
    _check(cfg, st, k0, outs[2], [(1, 2, 0), (0, 6, 3)], 1e-4)


def test_feeds_the_sentence_scores():
    """The output is accepted as the tok_redundancy input of the step and matches the oracle's
    step run with the oracle's R."""
    from helpers import compare_head, oracle_head, run_step
    cfg = W.CONFIGS[1].scaled(dtype="bf16")
    st = W.make_structure(cfg)
    k0, v0, q = W.fill_cache(cfg, st, device="cuda")
    red = _run(cfg, st, k0)
    k, v = k0.clone(), v0.clone()
    out = run_step(cfg, st, k, v, q, red=red)
    assert int(out.dev_status.item()) == 0
    stats = {}
    for h in range(cfg.n_kv_heads):
        red_o = torch.from_numpy(oracle.token_redundancy(k0[0, h].to(torch.float64).cpu().numpy())).reshape(1, 1, -1)
        full = torch.zeros((1, cfg.n_kv_heads, st.total_tokens), dtype=torch.float64)
        full[0, h] = red_o[0, 0]
        ora = oracle_head(cfg, st, k0, v0, q, 0, h, 0, red=full)
        compare_head(cfg, st, out, k, v, k0, v0, ora, 0, h, 0, stats)


def test_rows_sixteen_megabytes_apart():
    # the widest pitch that whole column blocks take 32-bit offsets for, and the first one that they do not
    lens = [66, 5, 130]
    st = _structure([[0, n] for n in lens])
    cfg = W.Config("tokred-pitch", 9, len(lens), 1, 1, 4, "bf16", 0, 0, 64, 8, 16, 16.0, 0.0)
    room = torch.empty((st.total_tokens * (1 << 23)), dtype=torch.bfloat16, device="cuda")
    g = torch.Generator(device="cuda")
    g.manual_seed(79)
    rows = torch.randn((st.total_tokens, 128), generator=g, device="cuda").to(torch.bfloat16)
    want = None
    for pitch in (128, (1 << 23) - 8, 1 << 23):
        k = room.as_strided((1, 1, st.total_tokens, 128), (8, 8, pitch, 1))
        k[0, 0] = rows
        out = _run(cfg, st, k)
        want = out if want is None else want
        assert torch.equal(out, want)
    _check(cfg, st, rows.view(1, 1, -1, 128), want, [(0, 0, b) for b in range(len(lens))], 1e-4)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("block_size", [1, 16, 24, 128])
def test_pages_give_the_bits_of_a_contiguous_cache(dtype, block_size):
    # rows of a column block are looked up a block ahead: lengths around blocks of 64 columns and workgroups of 256 rows
    from test_gpu_paged import _to_pages
    lens = [1, 63, 64, 65, 127, 128, 129, 191, 193, 255, 256, 257, 319, 321, 700]
    st = _structure([[0, n] for n in lens])
    cfg = W.Config("tokred-pages", 9, len(lens), 2, 3, 12, dtype, 0, 0, 64, 8, 16, 16.0, 0.0)
    g = torch.Generator(device="cuda")
    g.manual_seed(block_size)
    k = torch.randn((2, 3, st.total_tokens, 128), generator=g, device="cuda").to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    want = _run(cfg, st, k)
    kp, vp, table = _to_pages(cfg, st, k, k, block_size, seed=3)
    so, sp, sf = (torch.from_numpy(x).cuda() for x in (st.seq_off, st.sent_ptr, st.sent_off))
    cache = B.PagedCache(kp, vp, table, cfg.n_q_heads, so, sp, sf, st.total_tokens, st.total_sentences)
    ws = torch.empty(B.skipkv_redundancy_paged_workspace_bytes(cache), dtype=torch.uint8, device="cuda")
    got = torch.full_like(want, float("nan"))
    B.skipkv_token_redundancy_paged(cache, got, None, ws)
    torch.cuda.synchronize()
    assert torch.equal(got, want)
