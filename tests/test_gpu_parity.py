"""GPU parity: the HIP path through the C ABI against the CPU oracle, head by head, on the
same seeded bits.  Sizes are chosen so that the oracle finishes in seconds while the work
still spans several chunks, tiles and a ragged tail."""
import numpy as np
import pytest
import torch

from paper_2512_07993_amd import workloads as W

from helpers import check_all_heads_on_gpu, compare_head, oracle_head, run_step, sample_heads

pytestmark = pytest.mark.gpu


def _run_and_compare(cfg, n_heads, fused=True, seed=0, flags=0, all_heads=False):
    st = W.make_structure(cfg)
    k0, v0, q = W.fill_cache(cfg, st, device="cuda")
    k, v = k0.clone(), v0.clone()
    print("running", cfg.name, "tokens", st.total_tokens, "sentences", st.total_sentences, flush=True)
    out = run_step(cfg, st, k, v, q, fused=fused, flags=flags)
    assert int(out.dev_status.item()) == 0
    stats = {}
    for (l, h, b) in sample_heads(cfg, st, n_heads, seed):
        ora = oracle_head(cfg, st, k0, v0, q, l, h, b)
        compare_head(cfg, st, out, k, v, k0, v0, ora, l, h, b, stats)
    if all_heads:  # definition-level checks of every head of the step, on the GPU
        stats["all_heads_checked"] = check_all_heads_on_gpu(cfg, st, out, k, v, k0, v0)
    print(cfg.name, stats, flush=True)
    assert stats.get("near_tie_heads", 0) <= max(1, stats["heads"] // 20)
    return stats


def test_config1_tiny_fp32_all_heads():
    _run_and_compare(W.CONFIGS[1], 8)


def test_config1_separate_calls_match_fused():
    _run_and_compare(W.CONFIGS[1], 8, fused=False)


def test_config2_llama8b_single_full_size():
    """Config 2 with all 32 layers: 16 heads against the oracle, all 256 heads against
    the definition-level checks."""
    stats = _run_and_compare(W.CONFIGS[2], 16, seed=2, all_heads=True)
    assert stats["all_heads_checked"] == 256


def test_config3_ragged_batch_one_layer():
    _run_and_compare(W.CONFIGS[3].scaled(n_layers=1, batch=6), 12)


def test_config4_qwen7b_gqa7_one_layer():
    _run_and_compare(W.CONFIGS[4].scaled(n_layers=1, batch=5), 10)


def test_config5_longcot_one_layer():
    _run_and_compare(W.CONFIGS[5].scaled(n_layers=1, batch=1), 3)


def test_two_pass_scan_matches_oracle():
    """The fallback scan (K read twice, no cross-workgroup wait), forced for every sequence."""
    from paper_2512_07993_amd import binding as B
    _run_and_compare(W.CONFIGS[3].scaled(n_layers=1, batch=4), 8, flags=B.FLAG_FORCE_TWO_PASS)
    _run_and_compare(W.CONFIGS[1], 4, flags=B.FLAG_FORCE_TWO_PASS)


def test_two_pass_scan_is_reproducible_bit_for_bit():
    """The forced two-pass step run twice on the same bits: all sums are taken in a fixed order, so lambda, scores
    and kept indices repeat exactly (runs of several chunks: test_gpu_two_pass.py)."""
    import torch
    from paper_2512_07993_amd import binding as B
    cfg = W.CONFIGS[3].scaled(n_layers=2, batch=4)
    st = W.make_structure(cfg)
    k0, v0, q = W.fill_cache(cfg, st, device="cuda")
    runs = []
    for _ in range(2):
        k, v = k0.clone(), v0.clone()
        out = run_step(cfg, st, k, v, q, flags=B.FLAG_FORCE_TWO_PASS)
        assert int(out.dev_status.item()) == 0
        runs.append((out, k, v))
    (a, ka, va), (b, kb, vb) = runs
    for name in ("sent_lambda", "sent_score", "tok_imp"):
        assert torch.equal(getattr(a, name).view(torch.int32), getattr(b, name).view(torch.int32)), name
    for name in ("sent_keep", "kept_idx", "new_len", "new_sent_off", "new_sent_cnt"):
        assert torch.equal(getattr(a, name), getattr(b, name)), name
    assert torch.equal(ka.view(torch.int16), kb.view(torch.int16)) and torch.equal(va.view(torch.int16), vb.view(torch.int16))


def test_single_pass_scan_is_reproducible_bit_for_bit():
    """The same for the single-pass scan: records are merged in item order whatever the order of arrival."""
    import torch
    cfg = W.CONFIGS[3].scaled(n_layers=2, batch=4)
    st = W.make_structure(cfg)
    k0, v0, q = W.fill_cache(cfg, st, device="cuda")
    runs = []
    for _ in range(2):
        k, v = k0.clone(), v0.clone()
        out = run_step(cfg, st, k, v, q)
        assert int(out.dev_status.item()) == 0
        runs.append((out, k, v))
    (a, ka, va), (b, kb, vb) = runs
    for name in ("sent_lambda", "sent_score", "tok_imp"):
        assert torch.equal(getattr(a, name).view(torch.int32), getattr(b, name).view(torch.int32)), name
    for name in ("sent_keep", "kept_idx", "new_len", "new_sent_off", "new_sent_cnt"):
        assert torch.equal(getattr(a, name), getattr(b, name)), name
    assert torch.equal(ka.view(torch.int16), kb.view(torch.int16)) and torch.equal(va.view(torch.int16), vb.view(torch.int16))


def test_bounded_wait_reports_timeout_and_those_heads_are_done_by_the_two_pass_scan():
    """With a poll limit below zero a workgroup that finds its head's statistics not ready gives up at
    once (the limit comes from the host: every kernel still runs to its normal end).  The step must
    complete and raise the time-out bit; every head that a time-out touched is flagged and done again by the
    two-pass kernels that follow the single-pass scan in the stream, so that all scores are valid, every
    head matches the oracle and is compacted by its own kept indices; and the library stays usable (the next
    call, with the default limit, is correct again)."""
    import torch
    from paper_2512_07993_amd import binding as B
    cfg = W.CONFIGS[3].scaled(n_layers=1, batch=4)
    st = W.make_structure(cfg)
    k0, v0, q = W.fill_cache(cfg, st, device="cuda")
    k, v = k0.clone(), v0.clone()
    out = run_step(cfg, st, k, v, q, spin_limit=-1)
    status = int(out.dev_status.item())
    assert status & B.DEV_TIMEOUT
    assert not (status & ~B.DEV_TIMEOUT), status
    assert not bool(torch.isnan(out.sent_score).any())
    stats = {}
    for (l, h, b) in sample_heads(cfg, st, 8, 3):
        ora = oracle_head(cfg, st, k0, v0, q, l, h, b)
        compare_head(cfg, st, out, k, v, k0, v0, ora, l, h, b, stats)
    assert check_all_heads_on_gpu(cfg, st, out, k, v, k0, v0) == cfg.n_layers * cfg.n_kv_heads * cfg.batch
    print("after time-outs:", stats, flush=True)
    _run_and_compare(cfg, 6)


def test_config3_full_size_sampled_heads():
    """The benchmark workload itself (all 32 layers, batch 16: the grid, plan and workspace sizes
    that bench.py times), checked on heads sampled across layers, heads and sequences."""
    stats = _run_and_compare(W.CONFIGS[3], 16, seed=3, all_heads=True)
    assert stats["heads"] == 16 and stats["all_heads_checked"] == 4096


def test_config4_full_size_sampled_heads():
    """Qwen-7B shape at full size (64 sequences, 28 layers, GQA 7, alpha 8) on sampled heads."""
    stats = _run_and_compare(W.CONFIGS[4], 12, seed=4, all_heads=True)
    assert stats["heads"] == 12 and stats["all_heads_checked"] == 7168


def test_config5_full_size_sampled_heads():
    """Long-CoT shape at full size (8 sequences of 32896 tokens, 48 layers, 160 query rows per head:
    the two-pass scan) on sampled heads."""
    stats = _run_and_compare(W.CONFIGS[5], 6, seed=5, all_heads=True)
    assert stats["heads"] == 6 and stats["all_heads_checked"] == 3072


def test_long_sequences_next_to_short_ones():
    """Sequences of up to 99 K tokens (about 210 scan items of four spans each, near the 256 that one head may
    have in the single-pass scan: every workgroup of such a head merges all of its records) in one launch
    with sequences a third as long."""
    cfg = W.CONFIGS[3].scaled(n_layers=1, batch=3, n_kv_heads=2, n_q_heads=8, len_lo=30000, len_hi=100000,
                              sent_mean=40.0)
    stats = _run_and_compare(cfg, 6, seed=7)
    assert stats["heads"] == 6


@pytest.mark.parametrize("group,alpha,dtype", [
    (1, 1, "bf16"), (1, 32, "bf16"), (2, 16, "bf16"), (3, 8, "bf16"), (4, 4, "f32"), (5, 8, "bf16"), (6, 10, "bf16"),
    (7, 8, "bf16"), (8, 8, "bf16"), (8, 4, "f32"), (4, 32, "bf16"), (8, 32, "bf16"), (5, 32, "f32"),
])
def test_group_sizes_and_observation_windows(group, alpha, dtype):
    """Every shape of the query block: group sizes 1-8, windows 1-32; up to 64 query rows the
    single-pass scan runs, beyond that the two-pass one.  All heads against the oracle."""
    cfg = W.Config("rows-%dx%d" % (group, alpha), 40 + group * 33 + alpha, 3, 1, 2, 2 * group, dtype, 150, 900, 256,
                   alpha, max(alpha, 40), 12.0, 0.2)
    stats = _run_and_compare(cfg, 6)
    assert stats["heads"] == 6


@pytest.mark.parametrize("group,alpha,flags_name", [(4, 16, ""), (7, 8, ""), (5, 32, ""), (4, 16, "two_pass")])
def test_logits_far_from_the_first_ones_take_the_exact_statistics(group, alpha, flags_name):
    """Keys that carry a large component along a fixed direction during every other stretch of 50 tokens, queries
    that point along it or against it: the logits of half the rows jump up by about 200 log2 units where such a
    stretch begins, those of the other half drop by as much.  The fixed reference that the scans take from a
    span's (or chunk's) first 16 tokens is then off by more than the exponent range of fp32 wherever a stretch
    begins later in the span (sums overflow; sums of the dropping rows vanish next to a jumping row of the
    same lane group), and those spans and chunks must be redone with exact references.  Everything is
    compared with the oracle as usual."""
    import torch
    from paper_2512_07993_amd import binding as B
    cfg = W.Config("jumps-%dx%d" % (group, alpha), 900 + group * 33 + alpha, 3, 1, 2, 2 * group, "bf16", 700, 2600, 384,
                   alpha, max(alpha, 40), 14.0, 0.2)
    st = W.make_structure(cfg)
    k0, v0, q = W.fill_cache(cfg, st, device="cuda")
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    u = torch.randn(128, generator=gen, device="cuda")
    u = u / u.norm()
    for b in range(cfg.batch):
        t0, t1 = int(st.seq_off[b]), int(st.seq_off[b + 1])
        ramp = 40.0 * ((torch.arange(t1 - t0, device="cuda") // 50) % 2).float()
        k0[:, :, t0:t1] = (k0[:, :, t0:t1].float() + ramp[None, None, :, None] * u).to(k0.dtype)
    sign = torch.ones(q.shape[2], q.shape[3], device="cuda")
    sign[(torch.arange(q.shape[2], device="cuda")[:, None] + torch.arange(q.shape[3], device="cuda")[None, :]) % 2 == 1] = -1.0
    q = (q.float() + 40.0 * sign[None, None, :, :, None] * u).to(q.dtype)
    k, v = k0.clone(), v0.clone()
    out = run_step(cfg, st, k, v, q, flags=B.FLAG_FORCE_TWO_PASS if flags_name else 0)
    assert int(out.dev_status.item()) == 0
    stats = {}
    for (l, h, b) in sample_heads(cfg, st, 6, 11):
        ora = oracle_head(cfg, st, k0, v0, q, l, h, b)
        compare_head(cfg, st, out, k, v, k0, v0, ora, l, h, b, stats)
    print(cfg.name, stats, flush=True)
    assert stats["heads"] == 6
