"""The work that a user of libskipkv has it do, as measurable cases.

A case is a dict of plain values: what is called ("kind"), the model's shape (layers, kv_heads, q_heads,
dtype), the batch (batch, len_lo, len_hi), the method's scalars (budget, obs, protect) and the text
(sent_mean, dup, long).  The kinds:

  step          skipkv_step: the first compression of sequences whose sentence ranges all heads share
  paged         the same on a paged cache, blocks of `block` token slots in random order
  decode        skipkv_step_ranges + skipkv_ranges_append: every later compression of a decode, when each
                head has a length and sentence ranges of its own: budget + about 128 new tokens go in, budget
                comes out, and the ranges that come out take the next 128 tokens
  decode_paged  the same on a paged cache
  tokens        the token-level flow: redundancy of every token, scores, token selection, compaction
  shared        the similarity taken from hidden states once for all heads, then scores, selection, compaction
  steer         the steering strength and the steering add of one decode step

Compaction rewrites K and V in place.  A serving process holds several batches and compresses each when it is
due, so a state holds two batches that take turns, and a window of recent queries that is another one at every
call, as it is in a decode (the same queries again would rank first what they ranked first before, and would
find their favourites at the front of the cache already).
"""
import math
import random

import torch

from paper_2512_07993_amd import binding as B

D = 128            # head dimension
N_BATCHES = 2      # batches that take turns
N_QUERIES = 5      # windows of recent queries that take turns
NEW_TOKENS = 128   # tokens decoded between two compressions


def _case(kind, **kw):
    c = dict(kind=kind, layers=32, kv_heads=8, q_heads=32, dtype="bf16", batch=1, len_lo=4096, len_hi=4096, budget=1024,
             obs=16, protect=64, sent_mean=20.0, dup=0.2, long=0.0, block=0, d_model=0)
    c.update(kw)
    return c


def listed():
    return [
        # the steering of every decode step of 64 samples, hidden size 3584: the smallest call there is
        dict(_case("steer", batch=64, d_model=3584), name="steer-64x3584"),
        # one layer, fp32: a call whose launches and latencies are all there is
        dict(_case("step", layers=1, dtype="f32", len_lo=1152, len_hi=1152, budget=1024, obs=8, protect=32,
                   sent_mean=16.0, dup=0.1), name="step-1layer-fp32"),
        # one user of an 8B model, budget 4096, right after 128 new tokens
        dict(_case("step", len_lo=4224, len_hi=4224, budget=4096, dup=0.15), name="step-8b-single"),
        # 16 users of an 8B model whose chains of thought are between 2 K and 16 K tokens long
        dict(_case("step", batch=16, len_lo=2048, len_hi=16384, budget=2048), name="step-8b-ragged16"),
        # 64 users of a 7B model with seven query heads for each KV head
        dict(_case("step", layers=28, kv_heads=4, q_heads=28, batch=64, len_lo=4096, len_hi=8192, budget=1024,
                   obs=8, protect=32, sent_mean=24.0, dup=0.25), name="step-7b-batch64"),
        # 32 K tokens of a 14B model: five query heads for each KV head and a window of 32: 160 query rows
        dict(_case("step", layers=48, kv_heads=8, q_heads=40, batch=4, len_lo=32896, len_hi=32896, budget=4096,
                   obs=32, protect=128, dup=0.3), name="step-14b-long"),
        # text with stretches that the segmentation does not cut (code, tables, formulas)
        dict(_case("step", batch=4, len_lo=3000, len_hi=9000, budget=2048, long=0.01), name="step-8b-unsegmented"),
        # the compression every 128 tokens from then on: 16 users, each head at budget + 128
        dict(_case("decode", batch=16, len_lo=2176, len_hi=2176, budget=2048), name="decode-8b-batch16"),
        # the same under a paged cache, as a serving engine keeps it: 64 users of the 7B model
        dict(_case("decode_paged", layers=28, kv_heads=4, q_heads=28, batch=64, len_lo=1152, len_hi=1152, budget=1024,
                   obs=8, protect=32, sent_mean=24.0, dup=0.25, block=16), name="decode-7b-paged64"),
        # the first compression under a paged cache
        dict(_case("paged", batch=8, len_lo=2048, len_hi=8192, budget=2048, block=16), name="paged-8b-ragged8"),
        # token-level scores and eviction: quadratic in the length
        dict(_case("tokens", batch=4, len_lo=2048, len_hi=4224, budget=2048), name="tokens-8b-ragged4"),
        # similarity from the hidden states, once for all heads
        dict(_case("shared", batch=8, len_lo=2048, len_hi=8192, budget=2048, d_model=4096), name="shared-8b-ragged8"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "step", "decode", "decode", "decode_paged", "paged", "tokens", "shared", "steer"])
    if kind == "steer":
        return _case("steer", batch=_log_int(rng, 1, 256), d_model=128 * rng.randint(7, 64) if rng.random() < 0.7 else rng.randint(900, 8192))
    kv, q = rng.choice([(8, 32), (8, 32), (4, 28), (8, 40), (8, 8), (2, 16), (4, 12)])
    obs = rng.choice([4, 8, 8, 16, 16, 32, rng.randint(3, 32)])
    c = _case(kind, layers=_log_int(rng, 1, 48), kv_heads=kv, q_heads=q, batch=_log_int(rng, 1, 64), obs=obs,
              protect=max(obs, rng.choice([32, 64, 128, rng.randint(32, 200)])), sent_mean=rng.choice([16.0, 20.0, 24.0, 31.0]),
              dup=round(rng.uniform(0.05, 0.3), 3), long=rng.choice([0.0, 0.0, 0.0, 0.01]))
    if kind in ("decode", "decode_paged"):
        c["budget"] = _log_int(rng, 512, 4096)
        c["len_lo"] = c["len_hi"] = c["budget"] + NEW_TOKENS
        c["batch"] = min(c["batch"], 32)
    else:
        a, b = _log_int(rng, 400, 24000), _log_int(rng, 400, 24000)
        if kind == "tokens":
            a, b = _log_int(rng, 400, 5000), _log_int(rng, 400, 5000)
        c["len_lo"], c["len_hi"] = min(a, b), max(a, b)
        c["budget"] = max(c["protect"] + 64, int((c["len_lo"] + c["len_hi"]) / 2 * rng.uniform(0.1, 0.9)))
    if "paged" in kind:
        c["block"] = rng.choice([16, 16, 32, 128])
    if kind == "shared":
        c["d_model"] = rng.choice([3584, 4096, 5120])
    if kind == "step" and rng.random() < 0.15 and q // kv <= 4:
        c.update(dtype="f32", obs=min(obs, 16), layers=min(c["layers"], 4), batch=min(c["batch"], 8))
    # no more than the largest listed case costs: fewer sequences, then fewer layers
    most = {"tokens": 4e6, "step": 20e6, "decode": 12e6, "decode_paged": 12e6}.get(kind, 8e6)
    if c["dtype"] == "f32":
        most = 1e6
    mean = (c["len_lo"] + c["len_hi"]) / 2
    while c["batch"] > 1 and c["batch"] * mean * c["layers"] * kv > most:
        c["batch"] = max(1, int(c["batch"] * 0.7))
    while c["layers"] > 1 and c["batch"] * mean * c["layers"] * kv > most:
        c["layers"] = max(1, int(c["layers"] * 0.7))
    return c


# ---- inputs ------------------------------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _lengths(case):
    """One length for each sequence, spread over the case's range, in an order of its own."""
    n, lo, hi = case["batch"], case["len_lo"], case["len_hi"]
    r = random.Random("%d %d %d" % (n, lo, hi))
    got = [min(hi, lo + int((b + r.random()) / n * (hi - lo + 1))) for b in range(n)]
    r.shuffle(got)
    return got


def _most_sentences(case, n):
    """More sentences than a text of n tokens has."""
    return min(n // 4 + 2, int(n / (0.6 * case["sent_mean"])) + 64)


def _sentences(case, n_tok, g):
    """Sentences of the rows (sequences, or heads of sequences) whose lengths are n_tok: offsets [rows, S + 1]
    (n_tok from the row's last sentence on), counts, and for every sentence the earlier one that it repeats (itself: none)
    and how closely.  Lengths are log-normal between 4 and 64 tokens; a share `long` of them has 129 to 400."""
    rows, cap = n_tok.numel(), _most_sentences(case, case["len_hi"])
    base = torch.empty(rows, cap, device="cuda").log_normal_(math.log(case["sent_mean"]) - 0.125, 0.5, generator=g).round().clamp(4, 64)
    if case["long"]:
        far = torch.rand(rows, cap, generator=g, device="cuda") < case["long"]
        base = torch.where(far, torch.randint(129, 401, (rows, cap), generator=g, device="cuda").to(base.dtype), base)
    at = torch.arange(cap, device="cuda").expand(rows, cap)
    again = torch.rand(rows, cap, generator=g, device="cuda") < case["dup"]
    root = torch.where(again, (torch.rand(rows, cap, generator=g, device="cuda") * at).floor().to(torch.int64).clamp(max=cap - 1), at)
    for _ in range(13):
        root = root.gather(1, root)
    off = torch.zeros(rows, cap + 1, dtype=torch.int64, device="cuda")
    off[:, 1:] = base.to(torch.int64).gather(1, root).cumsum(1)
    off = torch.minimum(off, n_tok[:, None])
    off[:, -1] = n_tok
    count = (off[:, :-1] < n_tok[:, None]).sum(1)
    # near-duplicates are not all equally near: their keys differ by 2 to 15 percent
    noise = torch.where(root != at, 0.02 + 0.13 * torch.rand(rows, cap, generator=g, device="cuda"), torch.zeros((), device="cuda"))
    return off, count, root, noise


def _repeats(off, root, noise, n_tok, row_start):
    """(destination, source, noise) of every token of a repeated sentence, as rows of the packed token axis."""
    top = int(n_tok.max())
    tok = torch.arange(top, device="cuda").expand(n_tok.numel(), top).contiguous()
    s = (torch.searchsorted(off, tok, right=True) - 1).clamp(max=root.shape[1] - 1)
    r = root.gather(1, s)
    src = off.gather(1, r) + tok - off.gather(1, s)
    hit = (r != s) & (tok < n_tok[:, None]) & (src < off.gather(1, s))
    dst = (row_start[:, None] + tok)[hit]
    return dst, (row_start[:, None] + src)[hit], noise.gather(1, s)[hit]


def _fill(t, repeats, g):
    """N(0, 1) rows, with the repeated sentences' rows near those that they repeat."""
    t.normal_(generator=g)
    if repeats is not None:
        dst, src, noise = repeats
        x = t[..., src, :].float()
        t[..., dst, :] = x.add_(torch.randn(x.shape, generator=g, device="cuda").mul_(noise[:, None])).to(t.dtype)


def _i32(t):
    return t.to(torch.int32).contiguous()


def _pools(case, n_tok, g):
    """Block table and, for every token slot of the packed axis, its block and its place in it."""
    bs = case["block"]
    nb = [-(-int(n) // bs) for n in n_tok]
    perm = torch.randperm(sum(nb), generator=g, device="cuda")
    table = torch.full((len(nb), max(nb)), -1, dtype=torch.int32, device="cuda")
    blk, slot, pos = [], [], 0
    for b, n in enumerate(nb):
        table[b, :n] = perm[pos:pos + n].to(torch.int32)
        t = torch.arange(int(n_tok[b]), device="cuda")
        blk.append(perm[pos + t // bs])
        slot.append(t % bs)
        pos += n
    return table, torch.cat(blk), torch.cat(slot), sum(nb)


def _batch(case, seed):
    """One batch: K and V with what describes them, queries, and the buffers that the calls fill."""
    g = _gen(seed)
    kind, L, H, Bn = case["kind"], case["layers"], case["kv_heads"], case["batch"]
    dt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    per_head = kind in ("decode", "decode_paged")
    st = {}
    n_tok = torch.tensor(_lengths(case), device="cuda")
    seq_off = torch.zeros(Bn + 1, dtype=torch.int64, device="cuda")
    seq_off[1:] = n_tok.cumsum(0)
    T = int(seq_off[-1])
    if per_head:
        # every head at its own length: up to a sentence below the budget, plus the new tokens
        cut = torch.randint(0, 24, (L * H * Bn,), generator=g, device="cuda")
        head_tok = n_tok.repeat(L * H) - cut
        off, count, root, noise = _sentences(case, head_tok, g)
        room = off.shape[1] - 1 + NEW_TOKENS // 8  # the new tokens bring sentences of their own
        sent_ptr = torch.arange(Bn + 1, device="cuda") * (room + 1)
        S = Bn * room
        head_off = torch.zeros(L, H, Bn, room + 1, dtype=torch.int32, device="cuda")
        head_off[..., :off.shape[1]] = off.view(L, H, Bn, -1)
        sent_off = head_off[0, 0].reshape(-1).contiguous()
        st["ranges"] = B.Ranges(_i32(head_tok).view(L, H, Bn), _i32(count).view(L, H, Bn), head_off.view(L, H, S + Bn))
        start = (torch.arange(L * H, device="cuda")[:, None] * T + seq_off[None, :-1]).reshape(-1)
        repeats = _repeats(off, root, noise, head_tok, start)
        st["n_new"] = torch.full((Bn,), NEW_TOKENS, dtype=torch.int32, device="cuda")
        nb = 6
        st["bnd_ptr"] = torch.arange(Bn + 1, dtype=torch.int32, device="cuda") * nb
        bnd = torch.rand(Bn, NEW_TOKENS, generator=g, device="cuda").argsort(1)[:, :nb].sort(1).values
        st["bnd_off"] = _i32(bnd).view(-1)
    else:
        off, count, root, noise = _sentences(case, n_tok, g)
        S = int(count.sum())
        sent_ptr = torch.zeros(Bn + 1, dtype=torch.int64, device="cuda")
        sent_ptr[1:] = (count + 1).cumsum(0)
        keep = torch.arange(off.shape[1], device="cuda")[None, :] <= count[:, None]
        sent_off = off[keep]
        repeats = _repeats(off, root, noise, n_tok, seq_off[:-1])
    so, sp, sf = _i32(seq_off), _i32(sent_ptr), _i32(sent_off)

    if "paged" in kind:
        table, blk, slot, n_blocks = _pools(case, n_tok, g)
        k = torch.zeros(L, n_blocks, case["block"], H, D, dtype=dt, device="cuda")
        v = torch.zeros_like(k)
        flat = torch.empty(L, H, T, D, dtype=dt, device="cuda")
        if per_head:
            _fill(flat.view(L * H * T, D), repeats, g)
        else:
            for l in range(L):
                _fill(flat[l], repeats, g)
        for l in range(L):
            k[l, blk, slot] = flat[l].transpose(0, 1)
            v[l].normal_(generator=g)
        del flat
        cache = B.PagedCache(k, v, table, case["q_heads"], so, sp, sf, T, S)
    else:
        k = torch.empty(L, H, T, D, dtype=dt, device="cuda")
        v = torch.empty(L, H, T, D, dtype=dt, device="cuda")
        if per_head:
            _fill(k.view(L * H * T, D), repeats, g)
            v.normal_(generator=g)
        else:
            for l in range(L):
                _fill(k[l], repeats, g)
                v[l].normal_(generator=g)
        cache = B.Cache(k, v, case["q_heads"], so, sp, sf, T, S)
    del repeats
    st["cache"] = cache
    st["q"] = [torch.randn(L, Bn, case["q_heads"], case["obs"], D, generator=g, device="cuda", dtype=dt) for _ in range(N_QUERIES)]
    if kind == "shared":
        # hidden states of the text: near-duplicate sentences are near here too
        hid = torch.randn(T, case["d_model"], generator=g, device="cuda", dtype=torch.bfloat16)
        dst, src, noise = _repeats(off, root, noise, n_tok, seq_off[:-1])
        x = hid[src].float()
        hid[dst] = x.add_(torch.randn(x.shape, generator=g, device="cuda").mul_(noise[:, None])).to(torch.bfloat16)
        st["hidden"] = hid
        st["shared_lambda"] = torch.zeros(S, dtype=torch.float32, device="cuda")
    st["stride"] = max(1, min(case["budget"], T))
    f = dict(dtype=torch.float32, device="cuda")
    i = dict(dtype=torch.int32, device="cuda")
    st["status"] = torch.zeros(1, **i)
    st["params"] = B.Params(case["obs"], case["protect"], case["budget"], dev_status=st["status"])
    # one array for all heads, with room for any text of these lengths
    most = S if per_head else sum(_most_sentences(case, int(n)) for n in n_tok)
    st["sent_score"] = torch.zeros(L * H * most, **f)
    st["sent_lambda"] = torch.zeros(L * H * most, **f)
    st["sent_keep"] = torch.zeros(L * H * most, dtype=torch.uint8, device="cuda")
    st["kept_idx"] = torch.zeros(L, H, Bn, st["stride"], **i)
    st["new_len"] = torch.zeros(L, H, Bn, **i)
    st["new_off"] = torch.zeros(L * H * (most + Bn), **i)
    st["new_cnt"] = torch.zeros(L, H, Bn, **i)
    if per_head:
        st["out_ranges"] = B.Ranges(st["new_len"], st["new_cnt"], st["new_off"])
    if kind == "tokens":
        for name in ("tok_imp", "tok_red", "tok_score"):
            st[name] = torch.zeros(L, H, T, **f)
    return st


def _ws_bytes(case, st):
    kind, cache, params = case["kind"], st["cache"], st["params"]
    if kind == "decode":
        return B.skipkv_ranges_workspace_bytes(cache, params)
    if kind == "decode_paged":
        return B.skipkv_ranges_paged_workspace_bytes(cache, params)
    if kind == "paged":
        return B.skipkv_paged_workspace_bytes(cache, params)
    n = B.skipkv_workspace_bytes(cache, params)
    if kind == "tokens":
        n = max(n, B.skipkv_redundancy_workspace_bytes(cache))
    if kind == "shared":
        n = max(n, B.skipkv_similarity_workspace_bytes(cache, case["d_model"]))
    return n


def prepare(case, seed):
    if case["kind"] == "steer":
        g = _gen(seed)
        rows, d = case["batch"], case["d_model"]
        return dict(kind="steer", hidden=torch.randn(rows, d, generator=g, device="cuda", dtype=torch.bfloat16),
                    vec=torch.randn(d, generator=g, device="cuda", dtype=torch.bfloat16),
                    n_nonexec=torch.randint(0, 20, (rows,), generator=g, device="cuda", dtype=torch.int32),
                    mask=(torch.rand(rows, generator=g, device="cuda") < 0.5).to(torch.uint8),
                    coef=torch.zeros(rows, dtype=torch.float32, device="cuda"))
    batches = [_batch(case, 1000003 * seed + j) for j in range(N_BATCHES)]
    need = max(_ws_bytes(case, st) for st in batches)
    return dict(kind=case["kind"], batches=batches, ws=torch.empty(need, dtype=torch.uint8, device="cuda"), calls=0)


# ---- one pass --------------------------------------------------------------------------------------

def run(state):
    kind = state["kind"]
    if kind == "steer":
        B.skipkv_steer_strength(state["n_nonexec"], 0.5, 0.02, state["coef"])
        B.skipkv_steer_add(state["hidden"], state["vec"], state["coef"], 0.0, state["mask"])
        return dict(hidden=state["hidden"], coef=state["coef"])
    st, ws = state["batches"][state["calls"] % N_BATCHES], state["ws"]
    q = st["q"][state["calls"] % N_QUERIES]
    state["calls"] += 1
    cache, params, stride = st["cache"], st["params"], st["stride"]
    scores = (st["sent_score"], st["sent_lambda"])
    kept = (st["kept_idx"], st["new_len"], st["new_off"], st["new_cnt"], stride)
    if kind == "step":
        B.skipkv_step(cache, params, q, None, *scores, None, st["sent_keep"], *kept, ws)
    elif kind == "paged":
        B.skipkv_step_paged(cache, params, q, None, *scores, None, st["sent_keep"], *kept, ws)
    elif kind == "decode":
        B.skipkv_step_ranges(cache, st["ranges"], params, q, None, *scores, None, st["sent_keep"], *kept, ws)
        B.skipkv_ranges_append(cache, st["out_ranges"], st["n_new"], st["bnd_ptr"], st["bnd_off"], st["status"])
    elif kind == "decode_paged":
        B.skipkv_step_ranges_paged(cache, st["ranges"], params, q, None, *scores, None, st["sent_keep"], *kept, ws)
        B.skipkv_ranges_append(cache, st["out_ranges"], st["n_new"], st["bnd_ptr"], st["bnd_off"], st["status"])
    elif kind == "tokens":
        B.skipkv_token_redundancy(cache, st["tok_red"], ws)
        B.skipkv_score(cache, params, q, st["tok_red"], *scores, st["tok_imp"], ws)
        B.skipkv_select_tokens(cache, params, st["tok_imp"], st["tok_red"], st["sent_lambda"], st["tok_score"], None, *kept)
        B.skipkv_compact(cache, st["kept_idx"], st["new_len"], stride)
    elif kind == "shared":
        B.skipkv_sentence_similarity(cache, st["hidden"], st["shared_lambda"], ws)
        B.skipkv_score_shared(cache, params, q, None, st["shared_lambda"], *scores, None, ws)
        B.skipkv_select(cache, params, st["sent_score"], st["sent_keep"], *kept)
        B.skipkv_compact(cache, st["kept_idx"], st["new_len"], stride)
    # K and V are rows moved bit for bit: compared as whole numbers
    bits = torch.int32 if cache.k.dtype == torch.float32 else torch.int16
    out = dict(sent_score=st["sent_score"], sent_lambda=st["sent_lambda"], kept_idx=st["kept_idx"], new_len=st["new_len"],
               new_off=st["new_off"], new_cnt=st["new_cnt"], k=cache.k.view(bits), v=cache.v.view(bits), status=st["status"])
    if kind == "tokens":
        out.update(tok_score=st["tok_score"], tok_imp=st["tok_imp"], tok_red=st["tok_red"])
    else:
        out["sent_keep"] = st["sent_keep"]
    return out


# ---- what a pass cannot do without --------------------------------------------------------------------

def work(case):
    if case["kind"] == "steer":
        n = case["batch"] * case["d_model"]
        return dict(bytes=2.0 * n + 2.0 * case["d_model"], flops=2.0 * n / 2)  # half of the rows, read and written
    e = 4 if case["dtype"] == "f32" else 2
    heads = case["layers"] * case["kv_heads"]
    lens = _lengths(case)
    group = case["q_heads"] // case["kv_heads"]
    tok = heads * sum(lens)
    sents = [n / case["sent_mean"] for n in lens]
    kept = heads * sum(min(case["budget"], n) for n in lens)
    # rows change place from the first evicted sentence on: all but the first few of a sequence that does not fit its budget
    moved = heads * sum(case["budget"] if n > case["budget"] else 0 for n in lens)
    byt = tok * D * e + 4.0 * moved * D * e                       # K once; K and V rows that move, read and written
    byt += case["layers"] * case["batch"] * case["q_heads"] * case["obs"] * D * e
    byt += 4.0 * kept + heads * sum(sents) * (4 + 4 + 1 + 4)      # kept indices; score, lambda, flag, new offset per sentence
    flops = 2.0 * tok * group * case["obs"] * D                   # every key against every query of its group's window
    if case["kind"] == "shared":
        byt += 2.0 * sum(lens) * case["d_model"]
        flops += sum(s * s for s in sents) * case["d_model"] + sum(lens) * case["d_model"]
    else:
        flops += tok * D + heads * sum(s * s for s in sents) * D  # sentence sums; pairs of sentences, each pair once
    if case["kind"] == "tokens":
        byt += tok * D * e + 3 * 4.0 * tok
        flops += heads * sum(n * n for n in lens) * D             # pairs of tokens, each pair once
    return dict(bytes=float(byt), flops=float(flops))


def tolerance(case):
    if case["kind"] == "steer":
        return "exact"  # one rounding of an exact sum
    # 32-bit sums of bf16 products.  The single-pass and the two-pass scan, which add in different orders, differ by
    # 3e-7 (2-norm) and 6e-6 (largest; cosines of unit vectors that carry 16 bits a component).  The ranking that
    # follows has ties that such differences decide: a sentence or token that changes sides shifts the rest of its
    # head's row, which was 0.2 percent of the whole values at most.
    return {"rel": 2e-6, "max": 3e-5, "differ": 0.01}
