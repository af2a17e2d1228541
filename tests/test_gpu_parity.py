"""HIP library vs CPU oracle, element by element, through the C ABI (needs an MI355X)."""
import json
import os

import numpy as np
import pytest

from paper_2605_01106_amd import workloads as W

pytestmark = pytest.mark.gpu

from oracle.hybrid_lm import HybridLM  # noqa: E402
from oracle.protocol import SpecDecoder  # noqa: E402
from parity_util import assert_close, run_lockstep, tolerances  # noqa: E402


@pytest.fixture(scope="module")
def B():
    from paper_2605_01106_amd import binding
    return binding


def _ctx(B, weights, batch, max_seq, kmax, G, **kw):
    return B.Context(weights, batch, max_seq, kmax, G, **kw)


def _say(tag):
    def f(w):
        print(f"[{tag}] rounds={w['rounds']} mean_n={w['mean_n']:.2f} min_gap={w['min_gap']:.2e} "
              f"err: logits={w['logits']:.2e} ssm={w['ssm']:.2e} conv={w['conv']:.2e} kv={w['kv']:.2e}", flush=True)
    return f


def test_c0_full_run(B):
    """Config 0 end to end: tiny fp32 hybrid, prompt 32, 64 new tokens, k = 2."""
    wl = W.WORKLOADS["c0"]
    seed = 1
    wts = W.make_weights(wl.cfg, seed)
    prompts = W.make_prompts(wl.cfg.vocab, 1, wl.prompt_len, seed)
    ctx = _ctx(B, wts, 1, 128, wl.k, wl.gen_len)
    w = run_lockstep(ctx, wts, prompts, [wl.prompt_len], wl.gen_len, wl.k, engine="step", min_gap=2e-5,
                     report=_say("c0"))
    assert w["rounds"] >= 20


@pytest.mark.parametrize("dtype", [W.F32, W.BF16])
def test_lively_ragged_batch(B, dtype):
    """Odd sizes, O(1) recurrence and attention (so state, window and cache errors move the
    logits), ragged prompts that span several prefill passes, several KV pages and tiles."""
    cfg = W.scaled_config("lively", n_layers=3, d_model=72, vocab=200, m_heads=3, m_head_dim=40, d_state=16,
                          n_q_heads=6, n_kv_heads=2, head_dim=24, d_ff=104, w_dtype=dtype)
    wts = W.make_lively_weights(cfg, 7)
    lens = [37, 5, 70, 18]
    prompts = W.make_prompts(cfg.vocab, 4, lens, 3)
    ctx = _ctx(B, wts, 4, 160, 4, 24, kv_page_tokens=16, prefill_chunk=16)
    run_lockstep(ctx, wts, prompts, lens, 24, 3, engine="pass", report=_say(f"lively-{dtype}"))


@pytest.mark.parametrize("dtype,heads,p,d_state,head_dim,page,chunk,overlap,lens", [
    (W.F32, 4, 12, 32, 32, 32, 32, 0, [97, 5, 64, 33, 1]),         # sequences that end with, within and before a pass; last pass of one position
    (W.BF16, 4, 64, 64, 32, 32, 40, 1, [80, 17, 41, 80, 3]),       # matmul-form scan, both branches on one stream
    (W.BF16, 3, 40, 16, 24, 16, 17, 0, [17, 34, 20, 9]),           # odd sizes, scalar attention and scan, the shortest packed pass
    (W.BF16, 4, 64, 128, 64, 64, 320, 0, [300, 40, 200, 96]),      # segmented scan, several row chunks of the attention
    (W.BF16, 4, 16, 64, 64, 32, 18, 2, [18, 1, 2, 36, 20, 35, 3])])   # last pass of 18 positions, three of seven sequences left
def test_packed_rows_of_ragged_prompts(B, dtype, heads, p, d_state, head_dim, page, chunk, overlap, lens):
    """Prefill passes over prompts of unequal length compute only the rows that exist, sequence behind sequence: states,
    caches, windows and logits of every sequence against the oracle, whatever its neighbours' lengths."""
    cfg = W.scaled_config("packed", n_layers=2, d_model=72, vocab=180, m_heads=heads, m_head_dim=p, d_state=d_state,
                          n_q_heads=4, n_kv_heads=2, head_dim=head_dim, d_ff=104, w_dtype=dtype)
    wts = W.make_lively_weights(cfg, 29)
    prompts = W.make_prompts(cfg.vocab, len(lens), lens, 8)
    ctx = _ctx(B, wts, len(lens), max(lens) + 40, 2, 8, kv_page_tokens=page, prefill_chunk=chunk, overlap_mode=overlap,
               kernel_flags=B.HH_KF_CANARIES)
    run_lockstep(ctx, wts, prompts, lens, 8, 2, engine="pass", report=_say(f"packed-{chunk}"))
    assert ctx.hh_check_canaries() == 0, B.hh_last_error(ctx.ctx)


@pytest.mark.parametrize("d_model,heads,d_ff,chunk,longest,others", [
    (1032, 16, 1536, 320, 300, [(150, 151, 299, 7), (20, 30, 9, 1), (300, 300, 300, 300)]),   # many rows, K splits of every product
    (264, 4, 320, 0, 20, [(3, 4, 1, 2), (19, 20, 18, 20), (20, 20, 20, 20)]),              # 100 rows planned, 30 of them there
    (520, 8, 104, 64, 60, [(10, 11, 12, 13), (59, 60, 1, 30), (60, 60, 60, 60)]),          # 300 planned, 106 there: the split's kernel
    (520, 8, 320, 24, 42, [(1, 25, 30, 42), (24, 3, 20, 10), (42, 42, 42, 42)])])          # two passes, the second of 90 rows at most
def test_bits_do_not_depend_on_the_other_prompts_lengths(B, d_model, heads, d_ff, chunk, longest, others):
    """The longest prompt of a batch gives the same bits whatever the lengths of the others: packing the rows that exist must
    not move a product to another kernel or K split."""
    cfg = W.scaled_config("alone", n_layers=2, d_model=d_model, vocab=180, m_heads=heads, m_head_dim=64, d_state=64,
                          n_q_heads=4, n_kv_heads=2, head_dim=64, d_ff=d_ff, w_dtype=W.BF16)
    wts = W.make_lively_weights(cfg, 31)
    first = W.make_prompts(cfg.vocab, 1, [longest], 9)[0]
    seen = []
    for lens in others:
        lens = [longest, *lens]
        prompts = W.make_prompts(cfg.vocab, len(lens), lens, 17 + lens[1])
        prompts[0, :longest] = first
        ctx = _ctx(B, wts, len(lens), longest + 12, 1, 4, prefill_chunk=chunk)
        ctx.hh_prefill(prompts, lens, 4)
        got = [ctx.hh_get_logits(2)[0]]
        for layer in range(cfg.n_layers):
            got += [a[0] for a in ctx.hh_get_state(layer)] + list(ctx.hh_get_kv(layer, 0, longest))
        seen.append(got)
    for other in seen[1:]:
        assert [np.array_equal(a, b) for a, b in zip(seen[0], other)] == [True] * len(got)


@pytest.mark.parametrize("batch,k,flags", [(3, 0, 0), (7, 1, 0), (16, 0, 0), (24, 0, 0), (48, 0, 0), (13, 4, 0), (80, 0, 0), (96, 0, 0),
                                           (40, 0, "HH_KF_MID_WIDE"), (30, 4, 0)])
def test_equal_prompts_give_equal_bits(B, batch, k, flags):
    """Every sequence of a batch of equal prompts gives the same bits: no row of a product is summed in another order than its
    neighbours (few rows, 4 to 16, 17 to 96 in both shapes, more)."""
    cfg = W.scaled_config("equal", n_layers=2, d_model=264, vocab=180, m_heads=4, m_head_dim=64, d_state=64,
                          n_q_heads=4, n_kv_heads=2, head_dim=64, d_ff=320, w_dtype=W.BF16)
    wts = W.make_lively_weights(cfg, 53)
    prompts = np.repeat(W.make_prompts(cfg.vocab, 1, [21], 3), batch, axis=0)
    ctx = _ctx(B, wts, batch, 64, k, 8, kernel_flags=getattr(B, flags) if flags else 0)
    ctx.hh_prefill(prompts, [21] * batch, 8)
    ctx.hh_draft(k)
    got = [ctx.hh_get_logits(2)] + ([ctx.hh_get_logits(0)] if k else [])
    ctx.hh_verify()
    got.append(ctx.hh_get_logits(1))
    ctx.hh_commit()
    got += [ctx.hh_get_state(layer)[0] for layer in range(cfg.n_layers)]
    assert [sum(not np.array_equal(a[0], a[b]) for b in range(batch)) for a in got] == [0] * len(got)


@pytest.mark.parametrize("k", [0, 1, 5])
def test_draft_lengths_and_plain_greedy(B, k):
    cfg = W.scaled_config("klen", n_layers=2, d_model=64, vocab=128, m_heads=2, m_head_dim=32, d_state=32,
                          n_q_heads=4, n_kv_heads=4, head_dim=16, d_ff=64, w_dtype=W.F32)
    wts = W.make_lively_weights(cfg, 11)
    lens = [9, 20]
    prompts = W.make_prompts(cfg.vocab, 2, lens, 5)
    ctx = _ctx(B, wts, 2, 96, 5, 16, prefill_chunk=8)
    run_lockstep(ctx, wts, prompts, lens, 16, k, engine="step", report=_say(f"k={k}"))


@pytest.mark.parametrize("k,d_state,dtype", [(2, 32, W.BF16), (4, 64, W.BF16), (8, 64, W.F32), (0, 128, W.BF16)])
def test_aligned_shapes_fast_paths(B, k, d_state, dtype):
    """Shapes whose rows are 16-byte aligned (heads and head dimension multiples of 4, state a
    multiple of 32) take the few-positions SSM kernel (8 or 16 lanes per state row, a partly
    filled last workgroup) and, with a bf16 cache and 32-token pages, the matrix-core attention
    with one to three 16-row tiles (k + 1 positions x 4 query heads per KV head); prompts straddle
    pages and key steps, one sequence finishes early."""
    cfg = W.scaled_config("aligned", n_layers=2, d_model=64, vocab=160, m_heads=4, m_head_dim=12, d_state=d_state,
                          n_q_heads=8, n_kv_heads=2, head_dim=32, d_ff=96, w_dtype=dtype)
    wts = W.make_lively_weights(cfg, 17)
    lens = [33, 6, 95]
    prompts = W.make_prompts(cfg.vocab, 3, lens, 21)
    ctx = _ctx(B, wts, 3, 160, 8, 30, kv_page_tokens=32, prefill_chunk=32)
    run_lockstep(ctx, wts, prompts, lens, 30, k, engine="pass", report=_say(f"aligned-k{k}-N{d_state}-{dtype}"))


@pytest.mark.parametrize("k,heads,p,batch,dtype", [(0, 8, 32, 1, W.F32), (2, 4, 20, 3, W.F32), (8, 8, 32, 2, W.BF16), (4, 32, 64, 20, W.F32)])
def test_state_size_16(B, k, heads, p, batch, dtype):
    """State size 16 on aligned shapes: 4 lanes per state row in the few-positions scan, a partly filled last workgroup
    (20 rows of a head), several row groups per wavefront in the rebuild and four wavefronts per workgroup (32 heads x 64)."""
    cfg = W.scaled_config("state16", n_layers=2, d_model=64, vocab=160, m_heads=heads, m_head_dim=p, d_state=16,
                          n_q_heads=4, n_kv_heads=2, head_dim=32, d_ff=96, w_dtype=dtype)
    wts = W.make_lively_weights(cfg, 37)
    lens = [(7 * b) % 31 + 4 for b in range(batch)]
    prompts = W.make_prompts(cfg.vocab, batch, lens, 5)
    ctx = _ctx(B, wts, batch, 96, 8, 12, prefill_chunk=8, kernel_flags=B.HH_KF_CANARIES)
    run_lockstep(ctx, wts, prompts, lens, 12, k, engine="pass", report=_say(f"state16-k{k}"))
    assert ctx.hh_check_canaries() == 0, B.hh_last_error(ctx.ctx)


@pytest.mark.parametrize("head_dim,n_q,page,k,lens,splits", [
    (64, 4, 16, 2, [30, 63, 64, 65, 130], 0),     # whole head dimensions: tiles that end at, before and behind a tile's last key
    (128, 2, 64, 8, [190, 12], 1),                # several tiles in one slice, the next requested while one is scored
    (256, 2, 32, 0, [140, 64, 3], 32),
    (40, 4, 16, 15, [70, 1, 33], 0)])             # part of a 64-wide head; pages shorter than a tile, the table's end within one
def test_float32_attention_tiles(B, head_dim, n_q, page, k, lens, splits):
    """Float32 caches: whole key tiles are requested whatever is cached of them, the first one before the position is known."""
    cfg = W.scaled_config("f32attn", n_layers=2, d_model=64, vocab=160, m_heads=2, m_head_dim=16, d_state=16,
                          n_q_heads=n_q, n_kv_heads=2, head_dim=head_dim, d_ff=96, w_dtype=W.F32)
    wts = W.make_lively_weights(cfg, 41)
    prompts = W.make_prompts(cfg.vocab, len(lens), lens, 6)
    ctx = _ctx(B, wts, len(lens), max(lens) + 10 + 2 * k + 2, k, 10, kv_page_tokens=page, prefill_chunk=24, attn_max_splits=splits,
               kernel_flags=B.HH_KF_CANARIES)
    run_lockstep(ctx, wts, prompts, lens, 10, k, engine="pass", report=_say(f"f32-attention-{head_dim}"))
    assert ctx.hh_check_canaries() == 0, B.hh_last_error(ctx.ctx)


@pytest.mark.parametrize("dtype,head_dim,page", [(W.F32, 8, 16), (W.F32, 56, 32), (W.F32, 72, 16), (W.F32, 96, 64), (W.F32, 120, 256),
                                                 (W.BF16, 8, 16), (W.BF16, 24, 16), (W.BF16, 64, 16)])
def test_key_tiles_of_odd_head_dimensions(B, dtype, head_dim, page):
    """Key tiles whose items do not divide evenly over the threads, place after place, in prefill passes over cached keys (the
    second and later passes of a prompt) and in verification: float32 caches, and bf16 caches with pages of 16 tokens."""
    cfg = W.scaled_config("places", n_layers=2, d_model=64, vocab=160, m_heads=2, m_head_dim=16, d_state=16,
                          n_q_heads=4, n_kv_heads=2, head_dim=head_dim, d_ff=96, w_dtype=dtype)
    wts = W.make_lively_weights(cfg, 47)
    lens = [150, 64, 21]
    prompts = W.make_prompts(cfg.vocab, len(lens), lens, 6)
    ctx = _ctx(B, wts, len(lens), max(lens) + 20, 2, 6, kv_page_tokens=page, prefill_chunk=40, kernel_flags=B.HH_KF_CANARIES)
    run_lockstep(ctx, wts, prompts, lens, 6, 2, engine="pass", report=_say(f"places-{head_dim}"))
    assert ctx.hh_check_canaries() == 0, B.hh_last_error(ctx.ctx)


@pytest.mark.parametrize("batch,k,d_ff", [(8, 0, 96), (9, 0, 96), (17, 0, 96), (8, 2, 96), (7, 4, 5008), (11, 2, 8192)])
def test_float32_rows_in_tiles(B, batch, k, d_ff):
    """Float32 products of many rows: tiles of 8 rows in one launch, the rest behind them, whole and partly filled last tiles,
    argmax partials of all tiles; rows of 5008 and 8192 columns, of which 5 and 3 fit the LDS; prefill of 100 and more rows."""
    cfg = W.scaled_config("f32rows", n_layers=1, d_model=72, vocab=170, m_heads=4, m_head_dim=16, d_state=16,
                          n_q_heads=4, n_kv_heads=2, head_dim=24, d_ff=d_ff, w_dtype=W.F32)
    wts = W.make_lively_weights(cfg, 61)
    lens = [12 + (5 * b) % 7 for b in range(batch)]
    prompts = W.make_prompts(cfg.vocab, batch, lens, 13)
    ctx = _ctx(B, wts, batch, 48, k, 5, prefill_chunk=16, kernel_flags=B.HH_KF_CANARIES)
    run_lockstep(ctx, wts, prompts, lens, 5, k, engine="pass", report=_say(f"f32-rows-{batch * (k + 1)}"))
    assert ctx.hh_check_canaries() == 0, B.hh_last_error(ctx.ctx)


# ---------------------------------------------------------------------------------------------
# Long caches on thin models: the key-slice paths of the matrix-core attention that the
# paper-shaped workloads take at their real prompt lengths (Section 3.3, verification phase: M_H
# attends over the whole prefix), at a cost the float64 oracle can afford.

def _thin(name, head_dim, n_q, n_kv, **kw):
    base = dict(n_layers=2, d_model=64, vocab=192, m_heads=4, m_head_dim=16, d_state=32, n_q_heads=n_q,
                n_kv_heads=n_kv, head_dim=head_dim, d_ff=96, w_dtype=W.BF16)
    base.update(kw)
    return W.scaled_config(name, **base)


def test_long_cache_ticket_merge(B):
    """Head dimension 64, one sequence, 1100 cached keys, 32-token pages: 35 key steps, so the
    verification attention runs 9 key slices per KV head whose partial results are merged inside the
    kernel by the workgroup that draws the last ticket (18 workgroups, 37 KB of partials per row
    chunk: under both limits of that path).  Prefill chunks of 256 positions run the multi-tile
    kernel over a growing cache."""
    cfg = _thin("thin-ticket", 64, 4, 2)
    wts = W.make_lively_weights(cfg, 47)          # seeds audited: top-1/top-2 gap 5.4e-3
    lens = [1100]
    prompts = W.make_prompts(cfg.vocab, 1, lens, 12)
    ctx = _ctx(B, wts, 1, 1100 + 40, 2, 12, kv_page_tokens=32, prefill_chunk=256)
    w = run_lockstep(ctx, wts, prompts, lens, 12, 2, engine="pass", chunk=64, min_gap=1e-3, report=_say("ticket-merge"))
    assert w["rounds"] >= 4


def test_long_cache_merge_kernel_batch16(B):
    """Head dimension 64 (two 32-wide key blocks), 16 sequences with 1900..2110 cached keys, k = 4:
    16 key slices x 32 (sequence, KV head) pairs = 512 workgroups, so the slices are merged by the
    separate merge kernel; the batch is ragged, so slices end at different steps per sequence.
    The oracle follows the longest and the shortest sequence."""
    cfg = _thin("thin-merge", 64, 8, 2)
    wts = W.make_lively_weights(cfg, 47)          # seeds audited: top-1/top-2 gap 3.4e-3
    lens = [2110 - 14 * i for i in range(16)]
    prompts = W.make_prompts(cfg.vocab, 16, lens, 13)
    ctx = _ctx(B, wts, 16, 2110 + 48, 4, 10, kv_page_tokens=64, prefill_chunk=128)
    w = run_lockstep(ctx, wts, prompts, lens, 10, 4, engine="pass", chunk=64, oracle_rows=[0, 15],
                     min_gap=1e-3, report=_say("merge-kernel-b16"))
    assert w["rounds"] >= 2


@pytest.mark.parametrize("overlap_mode", [1, 3])
def test_long_cache_head128_three_row_tiles(B, overlap_mode):
    """Head dimension 128, 5 query heads per KV head, k = 8: 45 query rows = three 16-row tiles per
    workgroup, the new keys appended and scored inside the kernel, 3 sequences of about 1150 cached
    keys (10 slices per KV head, 245 KB of partials per row chunk: the separate merge kernel, as at
    the 3B shape).  Forced accepted counts exercise the rollback to every position.  Run once with the
    attention branch in line (overlap_mode 1) and once forked to the side stream beside the SSM
    branch in every pass (overlap_mode 3): the schedule must not change a result."""
    cfg = _thin("thin-h128", 128, 10, 2)
    wts = W.make_lively_weights(cfg, 41)          # seeds audited: top-1/top-2 gap 8.2e-4
    lens = [1150, 1101, 1127]
    prompts = W.make_prompts(cfg.vocab, 3, lens, 14)
    forced = W.make_forced_pattern(32, 3, 8, 0.68, 3)
    ctx = _ctx(B, wts, 3, 1150 + 80, 8, 27, kv_page_tokens=64, prefill_chunk=192, overlap_mode=overlap_mode)
    w = run_lockstep(ctx, wts, prompts, lens, 27, 8, forced=forced, engine="pass", chunk=64,
                     min_gap=4e-4, report=_say(f"h128-rt3-overlap{overlap_mode}"))
    assert w["rounds"] >= 3


@pytest.mark.parametrize("max_splits,single", [(1, 0), (3, -1), (32, -1)])
def test_key_slices_do_not_change_results(B, max_splits, single):
    """The number of key slices is a tunable: one slice, three, and as many as the cache allows
    (split from the first step on), on caches of 70..200 keys with 32-token pages."""
    cfg = _thin("thin-slices", 32, 8, 2, d_state=64)
    wts = W.make_lively_weights(cfg, 42)          # seeds audited: top-1/top-2 gap 2.6e-3
    lens = [200, 70, 131]
    prompts = W.make_prompts(cfg.vocab, 3, lens, 15)
    ctx = _ctx(B, wts, 3, 256, 4, 12, kv_page_tokens=32, prefill_chunk=64, attn_max_splits=max_splits,
               attn_single_slice_steps=single)
    run_lockstep(ctx, wts, prompts, lens, 12, 3, engine="pass", min_gap=1e-3, report=_say(f"slices-{max_splits}"))


@pytest.mark.parametrize("flag", ["HH_KF_ATTN_SCALAR", "HH_KF_SSM_GENERAL", "HH_KF_MID_OFF", "HH_KF_SKINNY_OFF",
                                  "HH_KF_SSM_SCALAR_CONV", "HH_KF_MID_OFF|HH_KF_ROWS_LDS", "HH_KF_NO_HANDOVER"])
def test_kernel_selection_flags_do_not_change_results(B, flag):
    """Every kernel-selection switch routes a family of launches to the slower kernel that computes
    the same thing; each variant is checked against the oracle on a workload that reaches the family:
    6 sequences with k = 3 give 6 draft rows (skinny), 24 verification rows (mid) and 6 x 32 = 192
    prefill rows (many-row GEMM), a bf16 cache with 32-token pages and aligned SSM shapes."""
    cfg = _thin("thin-flags", 32, 4, 2, d_model=96, d_ff=160, d_state=32)
    wts = W.make_lively_weights(cfg, 46)          # seeds audited: top-1/top-2 gap 8.9e-4
    lens = [61, 33, 90, 47, 75, 52]
    prompts = W.make_prompts(cfg.vocab, 6, lens, 16)
    bits = 0
    for name in flag.split("|"):
        bits |= getattr(B, name)
    ctx = _ctx(B, wts, 6, 128, 3, 10, kv_page_tokens=32, prefill_chunk=32, kernel_flags=bits)
    run_lockstep(ctx, wts, prompts, lens, 10, 3, engine="pass", min_gap=4e-4, report=_say(flag))


def test_mid_rows_long_k_and_wide_head(B):
    """17..96 activation rows through the K-loop kernel with several K windows per workgroup:
    d_model 320 (2.5 windows of 128 columns, so the last window is partly outside K) and a
    24000-row LM head (enough weight tiles that a workgroup walks two windows: the loop, its
    tail and the K-chunk reduction); 5 sequences, k = 4: 25 rows in verification, 80 in the
    prefill passes, 5 in the draft steps."""
    cfg = W.scaled_config("midk", n_layers=2, d_model=320, vocab=24000, m_heads=4, m_head_dim=40, d_state=16,
                          n_q_heads=4, n_kv_heads=2, head_dim=32, d_ff=520, w_dtype=W.BF16)
    wts = W.make_lively_weights(cfg, 37)          # seeds audited: top-1/top-2 gap 2.5e-4
    lens = [40, 9, 70, 23, 33]
    prompts = W.make_prompts(cfg.vocab, 5, lens, 7)
    ctx = _ctx(B, wts, 5, 128, 4, 16, kv_page_tokens=32, prefill_chunk=16)
    run_lockstep(ctx, wts, prompts, lens, 16, 4, engine="pass", report=_say("midk"))


@pytest.mark.parametrize("keep_logits", [1, 0])
def test_row_block_kernel_chunks_planes_and_argmax(B, keep_logits):
    """17..96 activation rows with a long, thin model (d_inner = d_ff = 2048 against d_model 64):
    the out and down projections have few weight tiles and a long K (many K chunks per product, norm
    scale from the chunks' sums of squares), 25 verification rows and 80-row prefill passes (two and
    five row tiles).  The LM head's argmax is raised with atomic maxima in the chunk reduction; with
    keep_logits = 0 no logits are written at all: tokens, counts, state and cache must still match."""
    cfg = W.scaled_config("rowblock", n_layers=2, d_model=64, vocab=200, m_heads=32, m_head_dim=64, d_state=16,
                          n_q_heads=4, n_kv_heads=2, head_dim=32, d_ff=2048, w_dtype=W.BF16)
    wts = W.make_lively_weights(cfg, 50)          # seeds audited: top-1/top-2 gap 7.3e-4
    lens = [40, 9, 70, 23, 33]
    prompts = W.make_prompts(cfg.vocab, 5, lens, 7)
    ctx = _ctx(B, wts, 5, 128, 4, 12, kv_page_tokens=32, prefill_chunk=16, keep_logits=keep_logits)
    run_lockstep(ctx, wts, prompts, lens, 12, 4, engine="pass", min_gap=4e-4, compare_logits=bool(keep_logits),
                 report=_say(f"rowblock-keep{keep_logits}"))
    if not keep_logits:
        with pytest.raises(B.HHError) as ei:
            ctx.hh_get_logits(1)
        assert ei.value.status == B.HH_ESTATE


def test_many_rows_lively(B):
    """More than 96 activation rows (10 sequences x 16-position prefill chunks = 160 rows: the
    tiled matrix-core GEMM over pre-split activations) on the initialisation with order-one
    activations, which amplifies any loss of precision in the projections: a two-term bf16 split
    of the activations there (16 mantissa bits) puts hundreds of logits outside the tolerance."""
    cfg = W.scaled_config("lively", n_layers=3, d_model=72, vocab=200, m_heads=3, m_head_dim=40, d_state=16,
                          n_q_heads=6, n_kv_heads=2, head_dim=24, d_ff=104, w_dtype=W.BF16)
    wts = W.make_lively_weights(cfg, 8)           # seeds audited: top-1/top-2 gap 1.1e-4
    lens = [37, 5, 70, 18, 44, 63, 29, 51, 12, 66]
    prompts = W.make_prompts(cfg.vocab, 10, lens, 4)
    ctx = _ctx(B, wts, 10, 160, 4, 24, kv_page_tokens=32, prefill_chunk=16)
    run_lockstep(ctx, wts, prompts, lens, 24, 3, engine="pass", report=_say("many-rows-lively"))


def _say_t(tag):
    def f(w):
        print(f"[{tag}] rounds={w['rounds']} mean_n={w['mean_n']:.2f} min_margin={w['min_margin']:.2e} "
              f"err: logits={w['logits']:.2e} ssm={w['ssm']:.2e} conv={w['conv']:.2e} kv={w['kv']:.2e}", flush=True)
    return f


@pytest.mark.parametrize("dtype,runs", [(W.F32, [(0.6, 59), (0.3, 10)]), (W.BF16, [(0.6, 21), (0.3, 32)])])
def test_stochastic_acceptance_lockstep(B, dtype, runs):
    """Temperature > 0 (Eq. 6): first token, draft draws, rejection tests, correction and bonus
    tokens equal the oracle's, decision by decision, with the same counter-based uniforms; the
    targets row has the oracle's form, and state, window and cache follow the committed stream.
    Odd vocabulary (203: ragged tail of the drawing kernel's 4-element groups).  Seeds audited:
    no decision within 1e-4 of flipping (a logit error e moves a CDF edge by at most e / T times the
    mass it touches; the measured logit errors are 1e-6 for float32 and, on single entries, up to
    1e-3 for bf16 storage).  One context runs temperature 0.6, then greedy, then temperature 0.3
    with another seed: the captured launch sequences must pick up the new parameters."""
    cfg = W.scaled_config("lively", n_layers=3, d_model=72, vocab=203, m_heads=3, m_head_dim=40, d_state=16,
                          n_q_heads=6, n_kv_heads=2, head_dim=24, d_ff=104, w_dtype=dtype)
    wts = W.make_lively_weights(cfg, 7)
    lens = [37, 5, 70, 18]
    prompts = W.make_prompts(cfg.vocab, 4, lens, 3)
    ctx = _ctx(B, wts, 4, 160, 4, 12, kv_page_tokens=16, prefill_chunk=16)
    streams = []
    for i, (T, seed) in enumerate(runs):
        w = run_lockstep(ctx, wts, prompts, lens, 12, 3, engine="pass", temperature=T, sample_seed=seed,
                         min_margin=1e-4, report=_say_t(f"stochastic-{dtype}-T{T}"))
        assert 0.0 < w["mean_n"] < 3.0            # both kept and rejected drafts occurred
        streams.append(w["tokens"])
        if i == 0:   # back to temperature 0 on the same context: the greedy stream again
            run_lockstep(ctx, wts, prompts, lens, 12, 3, engine="pass", report=_say("greedy-after-stochastic"))
    assert streams[0] != streams[1]


def test_stochastic_wide_vocabulary_and_plain_sampling(B):
    """A 24001-entry vocabulary (every wavefront of the drawing workgroup walks its segment in
    several 256-entry groups, ragged end) with float32 weights, few decisions: the CDF edges are
    4e-5 apart, the audited seed keeps 8e-6 from the nearest one, the float32 logit error of 2e-6
    moves an edge by at most 4e-6 at T = 0.5.  Then k = 0: plain sampling from M_H."""
    cfg = W.scaled_config("widev", n_layers=1, d_model=64, vocab=24001, m_heads=2, m_head_dim=32, d_state=16,
                          n_q_heads=2, n_kv_heads=1, head_dim=32, d_ff=64, w_dtype=W.F32)
    wts = W.make_lively_weights(cfg, 3)
    lens = [11, 6]
    prompts = W.make_prompts(cfg.vocab, 2, lens, 2)
    ctx = _ctx(B, wts, 2, 64, 2, 4, prefill_chunk=8)
    run_lockstep(ctx, wts, prompts, lens, 4, 2, engine="pass", temperature=0.5, sample_seed=327, min_margin=8e-6,
                 report=_say_t("stochastic-wide"))
    cfg = W.scaled_config("klen", n_layers=2, d_model=64, vocab=128, m_heads=2, m_head_dim=32, d_state=32,
                          n_q_heads=4, n_kv_heads=4, head_dim=16, d_ff=64, w_dtype=W.F32)
    wts = W.make_lively_weights(cfg, 5)
    lens = [9, 21]
    prompts = W.make_prompts(cfg.vocab, 2, lens, 2)
    ctx = _ctx(B, wts, 2, 96, 5, 12, prefill_chunk=8)
    run_lockstep(ctx, wts, prompts, lens, 12, 0, engine="step", temperature=0.8, sample_seed=27, min_margin=4e-4,
                 report=_say_t("plain-sampling"))


def test_stochastic_call_rules(B):
    """At temperature > 0 replaced drafts and forced counts are refused (neither has a draft
    distribution or a correction token); a bad temperature is refused; sampling cannot change
    inside a round."""
    import torch
    cfg = W.scaled_config("rules", n_layers=1, d_model=64, vocab=96, m_heads=2, m_head_dim=32, d_state=16,
                          n_q_heads=2, n_kv_heads=1, head_dim=32, d_ff=64, w_dtype=W.F32)
    wts = W.make_lively_weights(cfg, 1)
    lens = [8, 5]
    prompts = W.make_prompts(cfg.vocab, 2, lens, 1)
    ctx = _ctx(B, wts, 2, 64, 2, 8, prefill_chunk=8)
    with pytest.raises(B.HHError):
        ctx.hh_set_sampling(-1.0, 0)
    with pytest.raises(B.HHError):
        ctx.hh_set_sampling(float("nan"), 0)
    ctx.hh_set_sampling(0.7, 3)
    ctx.hh_prefill(prompts, lens, 8)
    ctx.hh_draft(2)
    with pytest.raises(B.HHError):
        ctx.hh_set_sampling(0.5, 3)
    with pytest.raises(B.HHError):
        ctx.hh_set_drafts(np.zeros((2, 2), np.int32))
    ctx.hh_verify()
    with pytest.raises(B.HHError):
        ctx.hh_commit(torch.zeros(2, dtype=torch.int32, device=ctx.device))
    ctx.hh_commit()
    d, g = ctx.hh_get_round()
    _, _, last_n = ctx.hh_get_lengths()
    for b in range(2):
        n = last_n[b]
        assert list(g[b][:n]) == list(d[b][:n]) and 0 <= g[b][n] < cfg.vocab and all(v == -1 for v in g[b][n + 1:])
        if n < 2:
            assert g[b][n] != d[b][n]


def test_draft_length_changes_every_round(B):
    """A different k every round on one context (the choice of k per round is the caller's: the
    adaptive draft length the paper names as future work needs nothing else from the library).
    Every round matches the oracle, and the committed stream equals that of a fixed k."""
    cfg = W.scaled_config("lively", n_layers=3, d_model=72, vocab=200, m_heads=3, m_head_dim=40, d_state=16,
                          n_q_heads=6, n_kv_heads=2, head_dim=24, d_ff=104, w_dtype=W.BF16)
    wts = W.make_lively_weights(cfg, 7)
    lens = [37, 5, 70, 18]
    prompts = W.make_prompts(cfg.vocab, 4, lens, 3)
    ctx = _ctx(B, wts, 4, 160, 4, 24, kv_page_tokens=16, prefill_chunk=16)
    w = run_lockstep(ctx, wts, prompts, lens, 24, [3, 0, 1, 4, 2], engine="pass", report=_say("k-schedule"))
    w2 = run_lockstep(ctx, wts, prompts, lens, 24, 3, engine="pass", report=_say("k-fixed"))
    assert w["tokens"] == w2["tokens"]


def test_forced_acceptance_and_arbitrary_drafts(B):
    """Forced accepted counts (drafts committed as drafted) and caller-supplied draft tokens."""
    cfg = W.scaled_config("forced", n_layers=2, d_model=64, vocab=96, m_heads=4, m_head_dim=16, d_state=8,
                          n_q_heads=2, n_kv_heads=1, head_dim=32, d_ff=128, w_dtype=W.BF16)
    wts = W.make_lively_weights(cfg, 13)
    lens = [12, 30, 7]
    prompts = W.make_prompts(cfg.vocab, 3, lens, 9)
    k, G = 4, 20
    forced = W.make_forced_pattern(64, 3, k, 0.6, 1)
    ctx = _ctx(B, wts, 3, 128, k, G, kv_page_tokens=32, prefill_chunk=32)
    run_lockstep(ctx, wts, prompts, lens, G, k, forced=forced, report=_say("forced"))
    override = W.make_random_drafts(cfg.vocab, 64, 3, k, 2)
    w = run_lockstep(ctx, wts, prompts, lens, G, k, override=override, report=_say("random-drafts"))
    # the committed stream does not depend on the draft source
    w2 = run_lockstep(ctx, wts, prompts, lens, G, k, report=_say("ssm-drafts"))
    assert w["tokens"] == w2["tokens"]


def test_graph_replay_matches_oracle(B):
    """With use_graphs the draft and verify launch sequences are captured on their second use and
    replayed afterwards; every replay (one per round, with read-backs and eager commits between
    them) is compared with the oracle, and the token stream with the eager run."""
    import torch
    wl = W.WORKLOADS["c0"]
    seed = 1
    wts = W.make_weights(wl.cfg, seed)
    prompts = W.make_prompts(wl.cfg.vocab, 1, wl.prompt_len, seed)
    eager = run_lockstep(_ctx(B, wts, 1, 128, wl.k, 40), wts, prompts, [wl.prompt_len], 40, wl.k, engine="step")
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        ctx = _ctx(B, wts, 1, 128, wl.k, 40, use_graphs=1)
        w = run_lockstep(ctx, wts, prompts, [wl.prompt_len], 40, wl.k, engine="step", report=_say("graphs"))
        # a second batch on the same context reuses the instantiated graphs
        w2 = run_lockstep(ctx, wts, prompts, [wl.prompt_len], 40, wl.k, engine="step", check_state_every=4)
    stream.synchronize()
    assert w["tokens"] == eager["tokens"] == w2["tokens"] and w["rounds"] >= 10


@pytest.mark.parametrize("dtype,d_state,chunk", [(W.F32, 64, 64), (W.F32, 128, 256), (W.BF16, 64, 128), (W.BF16, 256, 40)])
def test_prefill_scan_matmul_form(B, dtype, d_state, chunk):
    """Prefill passes of 16 and more positions take the matmul (state-space dual) form of the scan on
    the matrix cores: head dimension 64, state sizes 64 / 128 / 256, passes of 40 to 256 positions
    (several 32-position chunks per pass, a ragged last chunk and a ragged last pass per sequence, a
    sequence shorter than one chunk), weights with order-one recurrence so that a wrong decay factor,
    a dropped intra-chunk term or a wrong carried state moves the logits.  The state after prefill,
    the conv window, the logits and every later round are compared with the sequential float64 oracle;
    the same run with the position-by-position kernel (HH_KF_SSM_SEQUENTIAL) gives the same tokens."""
    cfg = W.scaled_config("ssd", n_layers=2, d_model=64, vocab=160, m_heads=4, m_head_dim=64, d_state=d_state,
                          n_q_heads=2, n_kv_heads=1, head_dim=32, d_ff=96, w_dtype=dtype)
    wts = W.make_lively_weights(cfg, 61)
    lens = [333, 17, 290, 97]
    prompts = W.make_prompts(cfg.vocab, 4, lens, 23)
    # (the library takes the matmul form by itself from 128 workgroups on; HH_KF_SSM_MATMUL forces it for these 4 x 2.  Rows
    # of the ring must be multiples of 16 bytes: head counts that are no multiple of 4 keep the sequential kernel)
    ctx = _ctx(B, wts, 4, 400, 3, 10, kv_page_tokens=32, prefill_chunk=chunk, kernel_flags=B.HH_KF_SSM_MATMUL)
    w = run_lockstep(ctx, wts, prompts, lens, 10, 3, engine="pass", chunk=64, report=_say(f"ssd-{dtype}-N{d_state}-T{chunk}"))
    seq = _ctx(B, wts, 4, 400, 3, 10, kv_page_tokens=32, prefill_chunk=chunk, kernel_flags=B.HH_KF_SSM_SEQUENTIAL)
    w2 = run_lockstep(seq, wts, prompts, lens, 10, 3, engine="pass", chunk=64)
    assert w["tokens"] == w2["tokens"]
    for c in (ctx, seq):
        c.hh_prefill(prompts, lens, 10)
    assert not np.array_equal(ctx.hh_get_state(0)[0], seq.hh_get_state(0)[0]), "same bits: the matmul form was not taken"


@pytest.mark.parametrize("dtype,d_state,heads,chunk", [(W.BF16, 64, 4, 96), (W.F32, 128, 4, 130), (W.BF16, 128, 32, 352),
                                                       (W.F32, 256, 28, 200), (W.BF16, 64, 4, 95)])
def test_prefill_scan_segments(B, dtype, d_state, heads, chunk):
    """Long passes over few sequences take the scan in segments: one chunk of 32 positions per segment (4 heads) and
    several (28 and 32 heads x 4 sequences), the shortest pass that takes the form (96 positions; 95 keeps the
    position-by-position kernel), passes that end inside a segment, sequences that end in the first, in a middle and in
    the last one or need no further pass.  Compared with the float64 oracle like the other forms, within the tolerance
    of the storage type; guard bytes behind every workspace region are checked."""
    cfg = W.scaled_config("seg", n_layers=2, d_model=64, vocab=160, m_heads=heads, m_head_dim=64, d_state=d_state,
                          n_q_heads=2, n_kv_heads=1, head_dim=32, d_ff=96, w_dtype=dtype)
    wts = W.make_lively_weights(cfg, 61)
    lens = [chunk + 101, 17, chunk - 40, 97]
    prompts = W.make_prompts(cfg.vocab, 4, lens, 23)
    ctx = _ctx(B, wts, 4, chunk + 160, 3, 8, kv_page_tokens=32, prefill_chunk=chunk, kernel_flags=B.HH_KF_CANARIES)
    run_lockstep(ctx, wts, prompts, lens, 8, 3, engine="pass", chunk=64, report=_say(f"seg-{dtype}-N{d_state}-H{heads}-T{chunk}"))
    assert ctx.hh_check_canaries() == 0
    seq = _ctx(B, wts, 4, chunk + 160, 3, 8, kv_page_tokens=32, prefill_chunk=chunk, kernel_flags=B.HH_KF_SSM_SEQUENTIAL)
    for c in (ctx, seq):
        c.hh_prefill(prompts, lens, 8)
    same = np.array_equal(ctx.hh_get_state(0)[0], seq.hh_get_state(0)[0])
    assert same == (chunk < 96), "the segments serve passes of 96 positions and more, and only those"


@pytest.mark.parametrize("d_state,heads,tokens", [(64, 4, 96), (128, 4, 128), (128, 4, 512), (256, 4, 320)])
def test_prefill_scan_segments_are_as_exact_as_the_sequential_scan(B, d_state, heads, tokens):
    """Distance of a float32 model's prefill from the float64 oracle: the scan in segments may be no further off than the
    position-by-position kernel.  Prompts are multiples of the 32-position chunk, so that the logits come from a position
    with a whole chunk's decays before it, and the decays are strong (log-decay sums of tens per chunk): decays taken as
    differences of float32 sums carry the rounding of sums that large (here 1.2 to 1.6 times the sequential kernel's
    distance for the logits, 1.9 to 3.6 times for the states).  With the sums in float64 the two forms only add the same
    products in another order: pooled over sequences and seeds the distances agree to 10 %, and 1.2 is the bound."""
    cfg = W.scaled_config("exact", n_layers=2, d_model=128, vocab=256, m_heads=heads, m_head_dim=64, d_state=d_state,
                          n_q_heads=2, n_kv_heads=1, head_dim=32, d_ff=96, w_dtype=W.F32)
    lens = [tokens] * 3
    off = {0: [0.0, 0.0], B.HH_KF_SSM_SEQUENTIAL: [0.0, 0.0]}
    for seed in (3, 4):
        wts = W.make_lively_weights(cfg, seed)
        prompts = W.make_prompts(cfg.vocab, 3, lens, seed)
        dec = SpecDecoder(HybridLM(cfg, wts.values), tokens + 8, engine="pass", chunk=64)
        dec.prefill([prompts[b] for b in range(3)], 2)
        for flags, sums in off.items():
            ctx = _ctx(B, wts, 3, tokens + 8, 1, 2, prefill_chunk=tokens, kernel_flags=flags)
            ctx.hh_prefill(prompts, lens, 2)
            got, ref = [ctx.hh_get_logits(2)], [np.array(dec.prefill_logits)]
            for layer in range(cfg.n_layers):
                got.append(ctx.hh_get_state(layer)[0])
                ref.append(np.array([st.S[layer] for st in dec.st]))
            for i, (g, r) in enumerate(zip(got, ref)):
                sums[min(i, 1)] += float(((g - r) ** 2).sum() / (r ** 2).sum())
    (logits, state), (logits_seq, state_seq) = (np.sqrt(v) for v in off.values())
    print(f"[exact-N{d_state}-T{tokens}] logits {logits:.2e} / {logits_seq:.2e}, states {state:.2e} / {state_seq:.2e}", flush=True)
    assert (logits, state) != (logits_seq, state_seq), "the two forms give the same bits: the segments were not taken"
    assert logits <= 1.2 * logits_seq and state <= 1.2 * state_seq


@pytest.mark.parametrize("form", ["segments", "walk", "sequential"])
def test_prefill_scan_with_decays_of_zero(B, form):
    """Decay rates beyond what float32 holds (exp(a_log) = inf: the state never outlives a step) and rates of 1e5, next to
    an ordinary head: every form of the prefill scan gives the oracle's finite results."""
    cfg = W.scaled_config("rates", n_layers=2, d_model=64, vocab=160, m_heads=4, m_head_dim=64, d_state=64,
                          n_q_heads=2, n_kv_heads=1, head_dim=32, d_ff=96, w_dtype=W.F32)
    wts = W.make_lively_weights(cfg, 12)
    for layer in range(cfg.n_layers):
        wts.put_vector(f"L{layer}.a_log", np.array([100.0, 12.0, 0.3, 95.0], np.float32))
    lens = [133, 60]
    prompts = W.make_prompts(cfg.vocab, 2, lens, 8)
    flags = {"segments": 0, "walk": B.HH_KF_SSM_MATMUL, "sequential": B.HH_KF_SSM_SEQUENTIAL}[form]
    ctx = _ctx(B, wts, 2, 160, 2, 8, prefill_chunk=128, kernel_flags=flags)
    run_lockstep(ctx, wts, prompts, lens, 8, 2, engine="step", report=_say(f"rates-{form}"))


@pytest.mark.parametrize("head_dim,n_q,n_kv,k,n", [(80, 4, 2, 15, 500), (128, 5, 1, 0, 777), (48, 4, 4, 8, 130), (32, 4, 2, 15, 300),
                                                   (128, 10, 2, 8, 420), (16, 2, 1, 4, 33), (200, 2, 2, 7, 400)])
def test_new_positions_in_the_attention_kernel(B, head_dim, n_q, n_kv, k, n):
    """The verification attention rotates, rounds and appends the new keys and values with all threads of the last
    slice and scores them from LDS: one to sixteen new positions (draft lengths from k = 15 down to 0, round by round: every
    fill of the two 8-position operand groups), head dimensions that fill the 32-wide operands (128, 32: one item per
    thread there), leave half of the last one empty (80, 48, 16) or keep the separate append (200: not a multiple of 16),
    positions that cross a page, one key slice and - at head dimension 128 from 13 key steps on - several, ragged prompts."""
    cfg = _thin("thin-new", head_dim, n_q, n_kv)
    wts = W.make_lively_weights(cfg, 47)
    lens = [n, n - 13, n // 2 + 1]
    prompts = W.make_prompts(cfg.vocab, 3, lens, 31)
    ctx = _ctx(B, wts, 3, n + 2 * k + 60, k, 2 * k + 12, kv_page_tokens=32, prefill_chunk=128, kernel_flags=B.HH_KF_CANARIES)
    worst = run_lockstep(ctx, wts, prompts, lens, 2 * k + 12, list(range(k, -1, -1)) if k == 15 else k, engine="pass", chunk=64,
                         report=_say(f"new-Dh{head_dim}-k{k}"))
    assert k < 15 or worst["rounds"] >= 16
    assert ctx.hh_check_canaries() == 0


@pytest.mark.parametrize("head_dim,n_q,n_kv,d_state,heads,batch,k", [
    (64, 6, 2, 128, 4, 1, 2), (128, 5, 1, 256, 4, 2, 4), (64, 16, 4, 128, 8, 16, 0), (96, 10, 2, 256, 8, 16, 8),
    (48, 8, 4, 256, 4, 3, 8), (128, 6, 2, 128, 4, 3, 1), (64, 5, 1, 256, 4, 2, 8)])
def test_both_branches_in_one_launch(B, head_dim, n_q, n_kv, d_state, heads, batch, k):
    """A pass of few positions runs attention and scan in one launch: against the oracle, and bit for bit against the two
    kernels on streams of their own, for one to nine positions, one to three row tiles, both operand widths, both lane counts
    per state row (16, and 8 with 16 sequences), one and several key slices, a page boundary crossed.  (The attention is wider
    than the state space, so that the output projections stay two launches on both sides: a pair may split its sums otherwise.)"""
    cfg = W.scaled_config("pair", n_layers=2, d_model=64, vocab=160, m_heads=heads, m_head_dim=64, d_state=d_state,
                          n_q_heads=n_q, n_kv_heads=n_kv, head_dim=head_dim, d_ff=96, w_dtype=W.BF16)
    wts = W.make_lively_weights(cfg, 23)
    lens = [max(150 - 31 * b, 30 + b) for b in range(batch)]
    prompts = W.make_prompts(cfg.vocab, batch, lens, 19)
    ks = [k, max(k - 1, 0), max(k - 3, 0)]
    G = 12
    run_lockstep(_ctx(B, wts, batch, 256, k, G, kernel_flags=B.HH_KF_CANARIES), wts, prompts, lens, G, ks, engine="pass",
                 chunk=64, report=_say(f"pair-{head_dim}-{d_state}-k{k}"))
    for splits in (1, 3):
        seen = []
        for overlap_mode in (1, 3):
            ctx = _ctx(B, wts, batch, 256, k, G, overlap_mode=overlap_mode, attn_max_splits=splits, attn_single_slice_steps=-1,
                       kernel_flags=B.HH_KF_CANARIES)
            ctx.hh_prefill(prompts, lens, G)
            got = []
            for kk in ks:
                ctx.hh_draft(kk)
                ctx.hh_verify()
                got.append(ctx.hh_get_logits(1))
                ctx.hh_commit()
            for layer in range(cfg.n_layers):
                got += list(ctx.hh_get_state(layer))
                for b in range(batch):
                    got += list(ctx.hh_get_kv(layer, b, ctx.hh_get_lengths()[0][b]))
            assert ctx.hh_check_canaries() == 0
            seen.append([a.tobytes() for a in got])
        assert seen[0] == seen[1]


@pytest.mark.parametrize("dtype,d_model,head_dim,n_q,m_heads,batch,ks", [
    (W.F32, 72, 24, 6, 5, 1, [2, 0]), (W.F32, 72, 40, 3, 5, 4, [0, 1]), (W.F32, 64, 64, 4, 8, 1, [5, 8]),     # 1, 3, 5, 8 rows and more
    (W.BF16, 1096, 64, 4, 24, 1, [2, 1, 0]), (W.BF16, 200, 32, 2, 66, 3, [0]),                  # 1..3 rows
    (W.BF16, 264, 64, 4, 24, 2, [1, 3, 6]), (W.BF16, 200, 48, 4, 44, 4, [2, 0]),                             # 4..16 rows
    (W.BF16, 264, 64, 4, 24, 5, [4, 7]), (W.BF16, 200, 48, 4, 36, 9, [1, 5, 8])])                           # 17..80 rows and more
def test_both_output_projections_in_one_launch(B, dtype, d_model, head_dim, n_q, m_heads, batch, ks):
    """The output projections of the two branches are one launch where both take the same kernel: every kernel family, rows of
    the attention's projection that end inside the split of the longer state-space rows (1 to 4 wavefronts of it have nothing
    to do), weight rows that leave the last tile or row group partly empty, row counts on both sides of every family's limits."""
    cfg = W.scaled_config("outs", n_layers=2, d_model=d_model, vocab=160, m_heads=m_heads, m_head_dim=32, d_state=32,
                          n_q_heads=n_q, n_kv_heads=1, head_dim=head_dim, d_ff=96, w_dtype=dtype)
    assert cfg.d_q <= cfg.d_inner
    wts = W.make_lively_weights(cfg, 29)
    lens = [34 - 3 * b for b in range(batch)]
    prompts = W.make_prompts(cfg.vocab, batch, lens, 21)
    ctx = _ctx(B, wts, batch, 128, max(ks), 14, overlap_mode=1, kernel_flags=B.HH_KF_CANARIES)
    run_lockstep(ctx, wts, prompts, lens, 14, ks, engine="pass", report=_say(f"outs-{dtype}-{d_model}-b{batch}"))
    assert ctx.hh_check_canaries() == 0


def _verification_launches(B, cfg, batch, k, **kw):
    """{kind of launch: count} of one verification pass of k + 1 positions."""
    wts = W.make_lively_weights(cfg, 23)
    lens = [30 + b % 7 for b in range(batch)]
    ctx = _ctx(B, wts, batch, 96, k, 12, **kw)
    ctx.hh_prefill(W.make_prompts(cfg.vocab, batch, lens, 19), lens, 12)
    ctx.hh_draft(k)
    ctx.hh_profile(True)
    ctx.hh_verify()
    seen = ctx.hh_profile_read()
    ctx.hh_profile(False)
    return {kind: n for (phase, kind), (n, _) in seen.items() if phase == 2}


ATTENTION, SCAN, OUT_PROJ, O_PROJ, BRANCHES, OUT_PROJS = 3, 1, 4, 5, 9, 10


@pytest.mark.parametrize("head_dim,n_q,n_kv,d_state,heads,batch,k,together", [
    # the shapes of test_both_branches_in_one_launch
    (64, 6, 2, 128, 4, 1, 2, True), (128, 5, 1, 256, 4, 2, 4, True), (64, 16, 4, 128, 8, 16, 0, True), (96, 10, 2, 256, 8, 16, 8, True),
    (48, 8, 4, 256, 4, 3, 8, True), (128, 6, 2, 128, 4, 3, 1, True), (64, 5, 1, 256, 4, 2, 8, True),
    # the last and the first behind each limit: workgroups of the scan with one and with two per compute unit, positions, row tiles,
    # head dimension, state size
    (128, 5, 1, 256, 8, 24, 4, True), (128, 5, 1, 256, 8, 25, 4, False), (64, 4, 2, 128, 32, 32, 0, True), (64, 4, 2, 128, 32, 33, 0, False),
    (64, 6, 2, 128, 4, 1, 9, False), (64, 16, 2, 128, 4, 1, 2, False), (64, 2, 2, 128, 4, 1, 5, False), (32, 4, 2, 128, 4, 1, 2, False),
    (136, 4, 2, 128, 4, 1, 2, False), (64, 6, 2, 64, 4, 1, 2, False)])
def test_which_passes_launch_both_branches_together(B, head_dim, n_q, n_kv, d_state, heads, batch, k, together):
    """The pass launches what the comparison of the two forms takes for granted, and apart what lies behind the rule's limits;
    what is timed are the launches of the pass."""
    cfg = W.scaled_config("pair", n_layers=2, d_model=64, vocab=160, m_heads=heads, m_head_dim=64, d_state=d_state,
                          n_q_heads=n_q, n_kv_heads=n_kv, head_dim=head_dim, d_ff=96, w_dtype=W.BF16)
    seen = _verification_launches(B, cfg, batch, k)
    assert (seen.get(BRANCHES, 0), seen.get(ATTENTION, 0), seen.get(SCAN, 0)) == ((2, 0, 0) if together else (0, 2, 2))


@pytest.mark.parametrize("dtype,d_model,head_dim,n_q,m_heads,batch,ks", [
    # the shapes of test_both_output_projections_in_one_launch; {k: whether the pass takes one launch}
    (W.F32, 72, 24, 6, 5, 1, {2: True, 0: True}), (W.F32, 72, 40, 3, 5, 4, {0: True, 1: True}), (W.F32, 64, 64, 4, 8, 1, {5: True, 7: True, 8: False}),
    (W.BF16, 1096, 64, 4, 24, 1, {2: True, 1: True, 0: True}), (W.BF16, 200, 32, 2, 66, 3, {0: True}),
    (W.BF16, 264, 64, 4, 24, 2, {1: True, 3: True, 6: True}), (W.BF16, 200, 48, 4, 44, 4, {2: True, 0: True}),
    (W.BF16, 264, 64, 4, 24, 5, {4: True, 7: True}), (W.BF16, 200, 48, 4, 36, 9, {1: True, 5: True, 8: False}),
    # attention rows longer than the state-space ones: apart up to 16 rows
    (W.BF16, 264, 64, 8, 4, 2, {0: False, 3: False, 8: True})])
def test_which_passes_launch_both_output_projections_together(B, dtype, d_model, head_dim, n_q, m_heads, batch, ks):
    cfg = W.scaled_config("outs", n_layers=2, d_model=d_model, vocab=160, m_heads=m_heads, m_head_dim=32, d_state=32,
                          n_q_heads=n_q, n_kv_heads=1, head_dim=head_dim, d_ff=96, w_dtype=dtype)
    for k, together in ks.items():
        seen = _verification_launches(B, cfg, batch, k, overlap_mode=1)
        assert (seen.get(OUT_PROJS, 0), seen.get(OUT_PROJ, 0), seen.get(O_PROJ, 0)) == ((2, 0, 0) if together else (0, 2, 2)), k


# (sequences, tokens, d_model, d_ff) of two-layer models and the plan (row tiles per wavefront, K splits) that each product
# of a prefill pass over all their rows gets: the input projection (in) and the attention's output (o) store, the
# state-space output (out) and the down projection add, gate/up (up) is the SwiGLU product
MANY_ROWS = [
    ((1, 97, 256, 96), {"in": (2, 1), "o": (2, 1), "out": (2, 1), "up": (2, 1), "down": (2, 1)}),
    ((1, 129, 512, 520), {"in": (2, 2), "o": (2, 1), "out": (2, 1), "up": (2, 2), "down": (2, 2)}),
    ((1, 400, 128, 5120), {"in": (2, 1), "o": (2, 1), "out": (2, 1), "up": (3, 1), "down": (2, 20)}),
    ((1, 400, 128, 6912), {"in": (2, 1), "o": (2, 1), "out": (2, 1), "up": (4, 1), "down": (2, 27)}),
    ((2, 801, 128, 2560), {"in": (2, 1), "o": (2, 1), "out": (2, 1), "up": (5, 1), "down": (2, 9)}),
    ((3, 897, 128, 4104), {"in": (2, 1), "o": (2, 1), "out": (2, 1), "up": (6, 1), "down": (3, 8)}),
    ((3, 897, 2560, 96), {"in": (3, 2), "o": (4, 1), "out": (4, 1), "up": (2, 5), "down": (4, 1)}),
    ((4, 801, 2560, 96), {"in": (5, 3), "o": (5, 1), "out": (5, 1), "up": (2, 5), "down": (5, 1)}),
    ((4, 1009, 2560, 96), {"in": (2, 1), "o": (6, 1), "out": (6, 1), "up": (2, 4), "down": (6, 1)}),
]


@pytest.mark.parametrize("d_model,head_dim,n_q,tokens", [
    (520, 24, 4, 260),      # one full and one almost empty group of 512 columns; 17 steps of 32 columns; 65 row tiles of the attention
    (1032, 128, 2, 271),    # three groups, held in registers
    (2048, 256, 2, 256),    # four groups, whole row tiles
    (2568, 64, 10, 300)])   # six groups: rows are read twice
def test_prefill_of_few_sequences(B, d_model, head_dim, n_q, tokens):
    """One prompt in one pass: split of rows of 1 to 6 groups of 512 columns with the norm, short tiles of the attention,
    products of odd numbers of steps."""
    cfg = W.scaled_config("fewseq", n_layers=1, d_model=d_model, vocab=160, m_heads=4, m_head_dim=64, d_state=64,
                          n_q_heads=n_q, n_kv_heads=2, head_dim=head_dim, d_ff=160, w_dtype=W.BF16)
    wts = W.make_lively_weights(cfg, 43)
    prompts = W.make_prompts(cfg.vocab, 1, [tokens], 4)
    ctx = _ctx(B, wts, 1, tokens + 20, 1, 4, prefill_chunk=512, kernel_flags=B.HH_KF_CANARIES)
    run_lockstep(ctx, wts, prompts, [tokens], 4, 1, engine="pass", report=_say(f"few-{d_model}"))
    assert ctx.hh_check_canaries() == 0, B.hh_last_error(ctx.ctx)


def _many_rows_model(d_model, d_ff):
    # two layers: the keys, values and state of the second one depend on every row of every product of the first
    return W.scaled_config("rows", n_layers=2, d_model=d_model, vocab=300, m_heads=4, m_head_dim=64, d_state=64,
                           n_q_heads=2, n_kv_heads=1, head_dim=32, d_ff=d_ff, w_dtype=W.BF16)


@pytest.mark.parametrize("shape,plans", MANY_ROWS)
def test_many_row_products_by_row_block(B, shape, plans):
    """The many-row products choose 64 to 192 activation rows per workgroup and a K split by a cost model: prefill passes
    of 97 to 4036 rows that reach every block height for the store, the residual add and SwiGLU, with a last block that is
    nearly empty, with and without a K split, with the SwiGLU result handed to the down projection and (d_ff no multiple of
    32, or a K split) without.  tests/test_many_row_plan.py checks that the plans are these and that they cover the
    kernel's shapes.  The second layer's keys and values attest every row of every product of the first one.  They may be
    off by their own 16-bit rounding (2^-9) and by a first-layer key that took the neighbouring 16-bit value: that moves a
    score by 2^-8 q k / sqrt(32), up to 0.03 where |q| and |k| are 6 (1.5 by design, four times that at the tail), and the
    attention's part of a row by as much - 3 % of the row's norm.  A row that misses a product or one of its K splits is
    off by 10 % and more."""
    sequences, tokens, d_model, d_ff = shape
    cfg = _many_rows_model(d_model, d_ff)
    wts = W.make_lively_weights(cfg, 5)
    lens = [tokens] * sequences
    prompts = W.make_prompts(cfg.vocab, sequences, lens, 9)
    dec = SpecDecoder(HybridLM(cfg, wts.values), tokens + 8, engine="pass", chunk=64)
    dec.prefill([prompts[b] for b in range(sequences)], 2)
    ctx = _ctx(B, wts, sequences, tokens + 8, 1, 2, prefill_chunk=tokens, kernel_flags=B.HH_KF_CANARIES)
    ctx.hh_prefill(prompts, lens, 2)
    assert_close("logits", ctx.hh_get_logits(2), np.array(dec.prefill_logits), *tolerances(cfg.w_dtype))
    worst = 0.0
    for layer in range(cfg.n_layers):
        for b in range(sequences):
            for got, ref in zip(ctx.hh_get_kv(layer, b, tokens), (dec.st[b].K[layer][:tokens], dec.st[b].V[layer][:tokens])):
                off = np.linalg.norm((got - ref).reshape(tokens, -1), axis=1) / np.linalg.norm(ref.reshape(tokens, -1), axis=1)
                worst = max(worst, float(off.max()))
    print(f"[rows-{shape}] worst key or value row off by {worst:.2e}", flush=True)
    assert worst < 0.03 and ctx.hh_check_canaries() == 0
