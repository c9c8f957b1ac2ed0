"""The compaction of calls whose kept rows may be so many that they are moved past the caches.  The host goes by the pitch of the index
list, the kernels by the rows that are kept: few of them in wide lists, and many, at every slice width that such calls have
and in steps of eight tiles."""
import numpy as np
import pytest
import torch

from paper_2512_07993_amd import binding as B
from paper_2512_07993_amd import workloads as W

from helpers import make_cache
from test_gpu_edges import _structure

pytestmark = pytest.mark.gpu


def _to_pages(k0, v0, n_toks, bs, g):
    nb = [-(-n // bs) for n in n_toks]
    perm = torch.randperm(sum(nb), generator=g, device="cuda").to(torch.int32)
    table = torch.full((2, max(nb)), -1, dtype=torch.int32, device="cuda")
    table[0, :nb[0]], table[1, :nb[1]] = perm[:nb[0]], perm[nb[0]:]
    t = [torch.arange(n, device="cuda") for n in n_toks]
    blk = torch.cat([table[b, t[b] // bs].long() for b in range(2)])
    slot = torch.cat([x % bs for x in t])
    kp = torch.zeros((k0.shape[0], sum(nb), bs, k0.shape[1], 128), dtype=k0.dtype, device="cuda")
    vp = torch.zeros_like(kp)
    kp[:, blk, slot], vp[:, blk, slot] = k0.transpose(1, 2), v0.transpose(1, 2)
    return kp, vp, table, blk, slot


# streams (16 a layer) and the slices that they are moved in: bf16 64 in steps, 512 of 128 bytes, 1024 of 256; fp32 128 in steps, 256 of 128,
# 512 of 256, 1024 of 512
@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("dtype,n_layers,n", [("bf16", 4, 13700), ("bf16", 32, 1730), ("bf16", 64, 870),
                                              ("f32", 8, 3430), ("f32", 16, 1730), ("f32", 32, 870), ("f32", 64, 440)])
def test_rows_moved_past_the_caches(dtype, n_layers, n, paged):
    H, n_toks, row = 4, [n + 90, n + 7], 256 if dtype == "bf16" else 512
    st = _structure([[0, x] for x in n_toks])
    T = st.total_tokens
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    k0, v0 = [torch.randn((n_layers, H, T, 128), generator=g, device="cuda").to(torch.bfloat16 if dtype == "bf16" else torch.float32) for _ in range(2)]
    rng = np.random.default_rng(n)
    kept = np.full((n_layers, H, 2, n), -1, np.int32)
    new_len = np.zeros((n_layers, H, 2), np.int32)
    for i, at in enumerate(np.ndindex(new_len.shape)):
        m = new_len[at] = (0, 1, 129, 300)[i // 23 % 4] if i % 23 == 5 else n - int(rng.integers(0, 40))  # some heads with few
        kept[at][:m] = np.sort(rng.choice(n_toks[at[2]], m, replace=False))
    assert 2 * row * int(new_len.sum()) > 200 << 20
    dk, dl = torch.from_numpy(kept).cuda(), torch.from_numpy(new_len).cuda()
    if paged:
        kp, vp, table, blk, slot = _to_pages(k0, v0, n_toks, 16, g)
        so, sp, sf = (torch.from_numpy(x).cuda() for x in (st.seq_off, st.sent_ptr, st.sent_off))
        cache = B.PagedCache(kp, vp, table, H, so, sp, sf, T, st.total_sentences)
        ws = torch.empty(B.skipkv_compact_paged_workspace_bytes(cache, n), dtype=torch.uint8, device="cuda")
        B.skipkv_compact_paged(cache, dk, dl, n, None, ws)
        k, v = kp[:, blk, slot].transpose(1, 2), vp[:, blk, slot].transpose(1, 2)
    else:
        cfg = W.Config("many", 9, 2, n_layers, H, H, dtype, 0, 0, 0, 1, 1, 1.0, 0.0)
        k, v = k0.clone(), v0.clone()
        B.skipkv_compact(make_cache(cfg, st, k, v), dk, dl, n)
    torch.cuda.synchronize()
    for l, h, b in np.ndindex(new_len.shape):
        t0, t1, m = int(st.seq_off[b]), int(st.seq_off[b + 1]), int(new_len[l, h, b])
        idx = torch.cat([dk[l, h, b, :m].long(), torch.arange(m, t1 - t0, device="cuda")]) + t0  # rows behind the kept ones are not written
        assert torch.equal(k[l, h, t0:t1], k0[l, h, idx]) and torch.equal(v[l, h, t0:t1], v0[l, h, idx]), (l, h, b)


@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("dtype,n_layers", [("bf16", 1), ("bf16", 17), ("bf16", 33), ("f32", 1), ("f32", 9), ("f32", 17), ("f32", 33)])
def test_few_rows_in_wide_index_lists(dtype, n_layers, paged):
    H, n_toks, bs = 4, [150, 300], 16
    st = _structure([[0, n] for n in n_toks])
    T = st.total_tokens
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device="cuda")
    g.manual_seed(n_layers)
    k0 = torch.randn((n_layers, H, T, 128), generator=g, device="cuda").to(dt)
    v0 = torch.randn((n_layers, H, T, 128), generator=g, device="cuda").to(dt)
    rng = np.random.default_rng(7)
    streams, row = 2 * n_layers * H * 2, 256 if dtype == "bf16" else 512
    stride = (200 << 20) // (streams * row) + 1
    kept = torch.full((n_layers, H, 2, stride), -1, dtype=torch.int32)
    new_len = torch.zeros((n_layers, H, 2), dtype=torch.int32)
    rows = {}
    for l in range(n_layers):
        for h in range(H):
            for b, n_tok in enumerate(n_toks):
                n = int(rng.choice([1, 16, 33, 64, 127, 129, n_tok - 1]))
                r = np.sort(rng.choice(n_tok, n, replace=False)).astype(np.int32)
                rows[l, h, b] = r
                kept[l, h, b, :n] = torch.from_numpy(r)
                new_len[l, h, b] = n
    kept, new_len = kept.cuda(), new_len.cuda()
    if paged:
        kp, vp, table, blk, slot = _to_pages(k0, v0, n_toks, bs, g)
        so, sp, sf = (torch.from_numpy(x).cuda() for x in (st.seq_off, st.sent_ptr, st.sent_off))
        cache = B.PagedCache(kp, vp, table, H, so, sp, sf, T, st.total_sentences)
        ws = torch.empty(B.skipkv_compact_paged_workspace_bytes(cache, stride), dtype=torch.uint8, device="cuda")
        B.skipkv_compact_paged(cache, kept, new_len, stride, None, ws)
        k, v = kp[:, blk, slot].transpose(1, 2), vp[:, blk, slot].transpose(1, 2)
    else:
        cfg = W.Config("stream", 9, 2, n_layers, H, H, dtype, 0, 0, 0, 1, 1, 1.0, 0.0)
        k, v = k0.clone(), v0.clone()
        B.skipkv_compact(make_cache(cfg, st, k, v), kept, new_len, stride)
    torch.cuda.synchronize()
    for (l, h, b), r in rows.items():
        t0, idx = int(st.seq_off[b]), torch.from_numpy(r).long().cuda() + int(st.seq_off[b])
        assert torch.equal(k[l, h, t0:t0 + len(r)], k0[l, h, idx]) and torch.equal(v[l, h, t0:t0 + len(r)], v0[l, h, idx])
