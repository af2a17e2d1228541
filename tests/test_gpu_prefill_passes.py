"""Prefill passes (needs an MI355X).  How a prompt is cut into passes is a schedule: the default (up to 4096 positions per sequence and
pass, 1024 of float32 models) gives what passes of 192 positions give, to rounding; the matmul-form scan gives what the sequential one gives."""
import numpy as np
import pytest

from paper_2605_01106_amd import workloads as W
from parity_util import assert_close, tolerances

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [W.BF16, W.F32])
@pytest.mark.parametrize("lens", [[4096 + 33], [2751, 2687, 64], [1025], [63, 1300, 1280, 1, 1215, 700]])   # (below, at and above a pass)
def test_default_passes(dtype, lens):
    from paper_2605_01106_amd import binding as B

    cfg = W.scaled_config("passes", n_layers=2, d_model=64, vocab=160, m_heads=2, m_head_dim=64, d_state=64, n_q_heads=2, n_kv_heads=1,
                          head_dim=32, d_ff=96, w_dtype=dtype)
    wts, prompts, n = W.make_lively_weights(cfg, 5), W.make_prompts(cfg.vocab, len(lens), lens, 4), len(lens)
    atol, rtol = tolerances(dtype)
    res = []
    for chunk in (0, 192):
        ctx = B.Context(wts, n, max(lens) + 24, 2, 8, kernel_flags=B.HH_KF_CANARIES, prefill_chunk=chunk)
        ctx.hh_prefill(prompts, lens, 8)
        out = [ctx.hh_get_logits(2)] + [v for layer in range(cfg.n_layers) for v in ctx.hh_get_state(layer)]
        out += [v for b in range(n) for v in ctx.hh_get_kv(cfg.n_layers - 1, b, lens[b])]
        ctx.hh_draft(2)
        ctx.hh_set_drafts(W.make_random_drafts(cfg.vocab, 1, n, 2, 2)[0])
        ctx.hh_verify()
        out.append(ctx.hh_get_logits(1)[:, 0])
        assert ctx.hh_get_lengths()[0] == lens and ctx.hh_check_canaries() == 0
        res.append(out)
        ctx.close()
    for i, (got, ref) in enumerate(zip(*res)):
        assert_close(f"output {i}", got, ref, atol, rtol, scale_to_ref=True)


@pytest.mark.parametrize("d_state,heads", [(64, 2), (64, 18), (128, 16), (256, 34)])   # (heads are shared out by 16)
def test_scan_inputs_shared_by_the_heads(d_state, heads):
    from paper_2605_01106_amd import binding as B

    cfg = W.scaled_config("shared", n_layers=2, d_model=64, vocab=160, m_heads=heads, m_head_dim=64, d_state=d_state, n_q_heads=2, n_kv_heads=1,
                          head_dim=32, d_ff=96, w_dtype=W.F32)
    lens = [97, 17, 33, 1, 64, 48, 80]        # passes of 48: chunks of 32 and 16, windows from the pass before, sequences that have ended
    wts, prompts = W.make_lively_weights(cfg, 6), W.make_prompts(cfg.vocab, len(lens), lens, 7)
    atol, rtol = tolerances(W.F32)
    res = []
    for flag in (B.HH_KF_SSM_MATMUL, B.HH_KF_SSM_SEQUENTIAL):
        ctx = B.Context(wts, len(lens), 130, 2, 8, prefill_chunk=48, kernel_flags=flag | B.HH_KF_CANARIES)
        ctx.hh_prefill(prompts, lens, 8)
        res.append([ctx.hh_get_logits(2)] + [v for layer in range(cfg.n_layers) for v in ctx.hh_get_state(layer)])
        assert ctx.hh_check_canaries() == 0
        ctx.close()
    for i, (got, ref) in enumerate(zip(*res)):
        assert_close(f"output {i}", got, ref, atol, rtol, scale_to_ref=True)


# at and above a pass, in the matmul-form scan: 4096 positions (one sequence; also at a width of 2048), 2560 (three), 1280 (six); 1024, 1024 and 672 in float32
@pytest.mark.parametrize("dtype,d_model,d_state,lens", [
    (W.BF16, 64, 64, [4096 + 33]), (W.BF16, 64, 128, [2561, 2560, 64]), (W.BF16, 64, 256, [1025]), (W.BF16, 64, 64, [63, 1300, 1280, 1, 1215, 700]),
    (W.BF16, 2048, 128, [4096 + 33]), (W.BF16, 2048, 64, [2048 + 1, 2048]),
    (W.F32, 64, 64, [2048 + 33]), (W.F32, 64, 256, [1025, 1024, 64]), (W.F32, 64, 128, [1025]), (W.F32, 64, 64, [63, 673, 672, 1, 660, 700])])
def test_passes_across_the_default_boundary(dtype, d_model, d_state, lens):
    from paper_2605_01106_amd import binding as B

    cfg = W.scaled_config("passes", n_layers=2, d_model=d_model, vocab=160, m_heads=4, m_head_dim=64, d_state=d_state, n_q_heads=2, n_kv_heads=1,
                          head_dim=32, d_ff=96, w_dtype=dtype)
    wts, prompts, n = W.make_lively_weights(cfg, 5), W.make_prompts(cfg.vocab, len(lens), lens, 4), len(lens)
    atol, rtol = tolerances(dtype)
    res = []
    for chunk in (0, 192):
        ctx = B.Context(wts, n, max(lens) + 24, 2, 8, kernel_flags=B.HH_KF_CANARIES, prefill_chunk=chunk)
        ctx.hh_prefill(prompts, lens, 8)
        out = [ctx.hh_get_logits(2)] + [v for layer in range(cfg.n_layers) for v in ctx.hh_get_state(layer)]
        out += [v for b in range(n) for v in ctx.hh_get_kv(cfg.n_layers - 1, b, lens[b])]
        ctx.hh_draft(2)
        ctx.hh_set_drafts(W.make_random_drafts(cfg.vocab, 1, n, 2, 2)[0])
        ctx.hh_verify()
        out.append(ctx.hh_get_logits(1)[:, 0])
        assert ctx.hh_get_lengths()[0] == lens and ctx.hh_check_canaries() == 0
        res.append(out)
        ctx.close()
    for i, (got, ref) in enumerate(zip(*res)):
        assert_close(f"output {i}", got, ref, atol, rtol, scale_to_ref=True)


@pytest.mark.parametrize("d_state,heads", [(64, 4), (64, 20), (128, 16), (256, 36)])   # (rows of 16 bytes only, so multiples of four; shared out by 16)
def test_scan_inputs_shared_by_the_heads_in_matmul_form(d_state, heads):
    from paper_2605_01106_amd import binding as B

    cfg = W.scaled_config("shared", n_layers=2, d_model=64, vocab=160, m_heads=heads, m_head_dim=64, d_state=d_state, n_q_heads=2, n_kv_heads=1,
                          head_dim=32, d_ff=96, w_dtype=W.F32)
    lens = [97, 17, 33, 1, 64, 48, 80]        # passes of 48: chunks of 32 and 16, windows from the pass before, sequences that have ended
    wts, prompts = W.make_lively_weights(cfg, 6), W.make_prompts(cfg.vocab, len(lens), lens, 7)
    atol, rtol = tolerances(W.F32)
    res = []
    for flag in (B.HH_KF_SSM_MATMUL, B.HH_KF_SSM_SEQUENTIAL):
        ctx = B.Context(wts, len(lens), 130, 2, 8, prefill_chunk=48, kernel_flags=flag | B.HH_KF_CANARIES)
        ctx.hh_prefill(prompts, lens, 8)
        res.append([ctx.hh_get_logits(2)] + [v for layer in range(cfg.n_layers) for v in ctx.hh_get_state(layer)])
        assert ctx.hh_check_canaries() == 0
        ctx.close()
    assert not np.array_equal(res[0][1], res[1][1])   # (two forms of the scan, not one compared with itself)
    for i, (got, ref) in enumerate(zip(*res)):
        assert_close(f"output {i}", got, ref, atol, rtol, scale_to_ref=True)


@pytest.mark.parametrize("flag", ["", "HH_KF_SSM_GENERAL", "HH_KF_SSM_SEQUENTIAL", "HH_KF_SSM_MATMUL", "HH_KF_SSM_SCALAR_CONV"])
@pytest.mark.parametrize("chunk,k", [(5, 2), (100, 8), (509, 4), (510, 2), (521, 13), (600, 28), (613, 8)])
def test_passes_longer_than_the_ring(flag, chunk, k):
    """Raw inputs of a pass: the window of the next pass, rollbacks across the end of a pass and the rounds behind them find theirs, whatever
    the pass length: up to 509 positions in a ring that holds the pass, from 510 on in two banks of 16 or 32 slots (the reference: passes of 480,
    held whole)."""
    from paper_2605_01106_amd import binding as B

    cfg = W.scaled_config("ring", n_layers=2, d_model=64, vocab=160, m_heads=4, m_head_dim=64, d_state=64, n_q_heads=2, n_kv_heads=1, head_dim=32,
                          d_ff=96, w_dtype=W.F32)
    lens = [3 * chunk - 1, 2 * chunk + 1, 2 * chunk + 2, 2 * chunk, chunk + 3, 1, chunk]
    wts, prompts, n = W.make_lively_weights(cfg, 8), W.make_prompts(cfg.vocab, len(lens), lens, 9), len(lens)
    atol, rtol = tolerances(W.F32)
    counts, drafts = np.random.default_rng(4).integers(0, k + 1, (3, n)).astype(np.int32), W.make_random_drafts(cfg.vocab, 3, n, k, 2)
    res = []
    for c in (chunk, 480):
        import torch
        ctx = B.Context(wts, n, 2000, k, 60, prefill_chunk=c, kernel_flags=(getattr(B, flag) if flag else 0) | B.HH_KF_CANARIES)
        ctx.hh_prefill(prompts, lens, 60)
        out = []
        for r in range(3):
            out += [v for layer in range(cfg.n_layers) for v in ctx.hh_get_state(layer)]
            ctx.hh_draft(k)
            ctx.hh_set_drafts(drafts[r])
            ctx.hh_verify()
            out.append(ctx.hh_get_logits(1)[:, 1:])
            ctx.hh_commit(torch.from_numpy(counts[r]).to("cuda:0"))
        assert ctx.hh_check_canaries() == 0
        res.append(out + [v for layer in range(cfg.n_layers) for v in ctx.hh_get_state(layer)])
        ctx.close()
    for i, (got, ref) in enumerate(zip(*res)):
        assert_close(f"output {i}", got, ref, atol, rtol, scale_to_ref=True)
