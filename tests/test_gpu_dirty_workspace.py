"""A call clears in its workspace what it counts in, in whichever kernel comes first: the same results, bit for bit, in a
workspace of ones as in one of zeros and in one that another call has just used."""
import numpy as np
import pytest
import torch

from paper_2512_07993_amd import binding as B
from paper_2512_07993_amd import workloads as W
from helpers import make_cache
from test_gpu_edges import _structure
from test_gpu_paged import _to_pages

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,bad_block", [("step", False), ("ranges", False), ("paged", False), ("paged", True), ("ranges_paged", False), ("ranges_paged", True)])
def test_results_do_not_depend_on_what_the_workspace_holds(kind, bad_block):
    L, H, group, alpha, budget, bs = 2, 2, 4, 8, 200, 16
    rng = np.random.default_rng(2)
    offsets = []
    for n in [700, 333, 90]:
        off = [0]
        while off[-1] < n:
            off.append(min(n, off[-1] + int(rng.integers(1, 40))))
        offsets.append(off)
    offsets[1] = [0, 20, 600, 650]  # (a sentence that the single-pass scan leaves to the two passes)
    st = _structure(offsets)
    cfg = W.Config("dirty", 9, 3, L, H, H * group, "bf16", 0, 0, budget, alpha, 32, 16.0, 0.0)
    g = torch.Generator(device="cuda")
    g.manual_seed(6)
    k0 = torch.randn((L, H, st.total_tokens, 128), generator=g, device="cuda").to(torch.bfloat16)
    q = torch.randn((L, 3, H * group, alpha, 128), generator=g, device="cuda").to(torch.bfloat16)
    results, ws = [], None
    for fill in (0, 255, None):
        status = torch.zeros(1, dtype=torch.int32, device="cuda")
        params = B.Params(alpha, 32, budget, dev_status=status)
        if "paged" in kind:
            kp, vp, table = _to_pages(cfg, st, k0, k0, bs, seed=4)
            if bad_block:  # (checked where the table is read: the sequence is flagged and left alone)
                table[2, 0] = 1 << 20
            so, sp, sf = (torch.from_numpy(x.astype(np.int32)).cuda() for x in (st.seq_off, st.sent_ptr, st.sent_off))
            cache = B.PagedCache(kp, vp, table, H * group, so, sp, sf, st.total_tokens, st.total_sentences)
        else:
            kp, vp = k0.clone(), k0.clone()
            cache = make_cache(cfg, st, kp, vp)
        S = st.total_sentences
        score = torch.zeros((L, H, S), device="cuda")
        lam = torch.zeros((L, H, S), device="cuda")
        keep = torch.zeros((L, H, S), dtype=torch.uint8, device="cuda")
        kept = torch.zeros((L, H, 3, 700), dtype=torch.int32, device="cuda")
        new_len, new_cnt = (torch.zeros((L, H, 3), dtype=torch.int32, device="cuda") for _ in range(2))
        new_off = torch.zeros((L, H, S + 3), dtype=torch.int32, device="cuda")
        ranges = B.Ranges(*[torch.from_numpy(x.astype(np.int32)).cuda().expand(L, H, x.size).contiguous() for x in (st.seq_len, st.n_sent, st.sent_off)])
        call, size = dict(step=(B.skipkv_step, B.skipkv_workspace_bytes), paged=(B.skipkv_step_paged, B.skipkv_paged_workspace_bytes),
                          ranges=(B.skipkv_step_ranges, B.skipkv_ranges_workspace_bytes),
                          ranges_paged=(B.skipkv_step_ranges_paged, B.skipkv_ranges_paged_workspace_bytes))[kind]
        if fill is not None:
            ws = torch.full((size(cache, params),), fill, dtype=torch.uint8, device="cuda")
        head = (cache, ranges, params) if "ranges" in kind else (cache, params)
        call(*head, q, None, score, lam, None, keep, kept, new_len, new_off, new_cnt, 700, ws)
        torch.cuda.synchronize()
        results.append([status, score.view(torch.int32), lam.view(torch.int32), keep, kept, new_len, new_off, new_cnt, kp, vp])
    assert (int(results[0][0]) != 0) == bad_block
    for other in results[1:]:
        for x, y in zip(results[0], other):
            assert torch.equal(x, y)
