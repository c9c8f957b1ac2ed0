"""The compaction of long chains of few streams, which moves 512 rows of a stream at a time: lengths around that, first moved
rows in front of and behind what one look for them covers (2048), heads that move nothing or too little for steps (up to 64 columns of
256 bytes and beyond 160: less than 1024 rows, in between: 2560), on both kinds of caches."""
import numpy as np
import pytest
import torch

from paper_2512_07993_amd import binding as B
from paper_2512_07993_amd import workloads as W

from helpers import make_cache
from test_gpu_edges import _structure

pytestmark = pytest.mark.gpu

STRIDE = 3000


def _kept(rng, n_tok, first, n):
    """n ascending rows, of which the first `first` stay where they are."""
    rest = np.sort(rng.choice(np.arange(first + 1, n_tok), n - first, replace=False)) if n > first else np.arange(0)
    return np.concatenate([np.arange(first), rest]).astype(np.int32)


@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("dtype,n_layers", [("bf16", 1), ("bf16", 2), ("bf16", 4), ("bf16", 8), ("f32", 1), ("f32", 2), ("f32", 4)])  # 32 to 256 columns of 256 bytes
def test_rows_moved_eight_tiles_at_a_time(dtype, n_layers, paged):
    H, n_toks, bs = 8, [4100, 3001], 16
    st = _structure([[0, n] for n in n_toks])
    T = st.total_tokens
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device="cuda")
    g.manual_seed(n_layers)
    k0 = torch.randn((n_layers, H, T, 128), generator=g, device="cuda").to(dt)
    v0 = torch.randn((n_layers, H, T, 128), generator=g, device="cuda").to(dt)
    rng = np.random.default_rng(11)
    shapes = [(0, 1), (0, 511), (0, 512), (0, 513), (3, 1027), (700, 701), (2047, 2500), (2048, 2049), (2100, 2900), (5, 3000), (40, 40), (0, 0),
              (511, 1024), (1, 1536), (2049, 2560), (0, 2048), (4, 1023), (4, 2559), (0, 2999)]
    kept = torch.full((n_layers, H, 2, STRIDE), -1, dtype=torch.int32)
    new_len = torch.zeros((n_layers, H, 2), dtype=torch.int32)
    rows = {}
    for l in range(n_layers):
        for h in range(H):
            for b, n_tok in enumerate(n_toks):
                first, n = shapes[(16 * l + 2 * h + b) % len(shapes)]
                r = rows[l, h, b] = _kept(rng, n_tok, first, n)
                kept[l, h, b, :n] = torch.from_numpy(r)
                new_len[l, h, b] = n
    new_len[0, 0, 0] = STRIDE + 1  # kept everything, more than its row of indices holds: left alone
    rows[0, 0, 0] = np.arange(0)
    kept, new_len = kept.cuda(), new_len.cuda()
    if paged:
        nb = [-(-n // bs) for n in n_toks]
        perm = torch.randperm(sum(nb), generator=g, device="cuda").to(torch.int32)
        table = torch.full((2, max(nb)), -1, dtype=torch.int32, device="cuda")
        table[0, :nb[0]], table[1, :nb[1]] = perm[:nb[0]], perm[nb[0]:]
        t = [torch.arange(n, device="cuda") for n in n_toks]
        blk = torch.cat([table[b, t[b] // bs].long() for b in range(2)])
        slot = torch.cat([x % bs for x in t])
        kp = torch.zeros((n_layers, sum(nb), bs, H, 128), dtype=dt, device="cuda")
        vp = torch.zeros_like(kp)
        kp[:, blk, slot], vp[:, blk, slot] = k0.transpose(1, 2), v0.transpose(1, 2)
        so, sp, sf = (torch.from_numpy(x).cuda() for x in (st.seq_off, st.sent_ptr, st.sent_off))
        cache = B.PagedCache(kp, vp, table, H, so, sp, sf, T, st.total_sentences)
        ws = torch.empty(B.skipkv_compact_paged_workspace_bytes(cache, STRIDE), dtype=torch.uint8, device="cuda")
        B.skipkv_compact_paged(cache, kept, new_len, STRIDE, None, ws)
        k, v = kp[:, blk, slot].transpose(1, 2), vp[:, blk, slot].transpose(1, 2)
    else:
        cfg = W.Config("steps", 9, 2, n_layers, H, H, dtype, 0, 0, 0, 1, 1, 1.0, 0.0)
        k, v = k0.clone(), v0.clone()
        B.skipkv_compact(make_cache(cfg, st, k, v), kept, new_len, STRIDE)
    torch.cuda.synchronize()
    for (l, h, b), r in rows.items():
        t0, t1 = int(st.seq_off[b]), int(st.seq_off[b + 1])
        idx = torch.cat([torch.from_numpy(r).long(), torch.arange(len(r), t1 - t0)]).cuda() + t0  # rows behind the kept ones are not written
        assert torch.equal(k[l, h, t0:t1], k0[l, h, idx]) and torch.equal(v[l, h, t0:t1], v0[l, h, idx]), (l, h, b)
