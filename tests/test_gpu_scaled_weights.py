"""The matrix cores meet bf16 weights as float16 tiles scaled by powers of two, and activations as two scaled float16 terms.
A model whose weights are multiplied by powers of two in ways that leave its function as it is shows that no scale is missed
and that none overflows or loses bits (needs an MI355X)."""
import copy

import numpy as np
import pytest
import torch

from paper_2605_01106_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2605_01106_amd import binding
    return binding


def _model(seed, d_ff=160, layers=2):
    # (head counts that put w_in, w_q, w_k and w_v on tiles of their own in the stacked projection)
    cfg = W.scaled_config("scaled", n_layers=layers, d_model=136, vocab=160, m_heads=16, m_head_dim=16, d_state=64, n_q_heads=4, n_kv_heads=2,
                          head_dim=32, d_ff=d_ff, w_dtype=W.BF16)
    return cfg, W.make_lively_weights(cfg, seed)


def _scale(wts, name, factor):
    put = wts.put_matrix if wts.values[name].ndim == 2 and not name.endswith("conv_w") else wts.put_vector
    put(name, (wts.values[name] * np.float32(1) * factor).astype(np.float32))


def _outputs(B, wts, batch, k, tokens):
    cfg = wts.cfg
    lens = [tokens - 3 * (b % 5) for b in range(batch)]
    prompts = W.make_prompts(cfg.vocab, batch, lens, 6)
    ctx = B.Context(wts, batch, tokens + 40, k, 12, kernel_flags=B.HH_KF_CANARIES)
    ctx.hh_prefill(prompts, lens, 12)
    out = [ctx.hh_get_logits(2)]
    ctx.hh_draft(k)
    if k:
        out.append(ctx.hh_get_logits(0)[:, :1])   # (the next rows follow tokens that a near tie may choose)
        ctx.hh_set_drafts(W.make_random_drafts(cfg.vocab, 1, batch, k, 2)[0])
    ctx.hh_verify()
    if k:
        out.append(ctx.hh_get_logits(1)[:, 1:])
    ctx.hh_commit(torch.zeros(batch, dtype=torch.int32, device="cuda:0"))
    out += [v for layer in range(cfg.n_layers) for v in ctx.hh_get_state(layer)]
    assert ctx.hh_check_canaries() == 0
    return out


SIZES = [(1, 2, 60), (1, 0, 400), (5, 0, 40), (12, 0, 60), (6, 2, 70), (10, 8, 50), (96, 0, 20), (16, 8, 30)]   # 3 to 1600 rows


@pytest.mark.parametrize("batch,k,tokens", SIZES)
def test_whole_matrices_times_powers_of_two(B, batch, k, tokens):
    """Norm weights, values and the up projection times 2^e, what they meet times 2^-e: every result is the same bits."""
    cfg, base = _model(3)
    for shift in (7, -20):
        scaled = copy.deepcopy(base)
        for i in range(cfg.n_layers):
            L = f"L{i}."
            for name, e in (("norm1", shift), ("w_in", -shift), ("w_q", -shift), ("w_k", -shift), ("w_v", -shift - 9), ("w_o", 9), ("gnorm", -shift),
                            ("w_out", shift), ("norm2", 2 * shift), ("w_gate", -2 * shift), ("w_up", -2 * shift + 15), ("w_down", -15)):
                _scale(scaled, L + name, 2.0 ** e)
        _scale(scaled, "final_norm", 2.0 ** shift)
        _scale(scaled, "lm_head", 2.0 ** -shift)
        for got, ref in zip(_outputs(B, scaled, batch, k, tokens), _outputs(B, base, batch, k, tokens)):
            assert np.isfinite(ref).all() and np.array_equal(got, ref)


@pytest.mark.parametrize("batch,k,tokens", SIZES)
def test_columns_times_powers_of_two(B, batch, k, tokens):
    """The same column by column, a range of 2^12 in one row of activations and its inverse in the weights: no factor of a column is
    missed.  What a cached key or value of the other 16-bit neighbour makes of float32 rounding is 2e-5 at most here.  (A power of two
    leaves a term's bits as they are, so a low term that is lost in both models alike does not show: the products against float64 are in
    test_gpu_product_accuracy.py.)"""
    cfg, base = _model(4, d_ff=96, layers=1)
    r = np.random.default_rng(1)
    scaled = copy.deepcopy(base)
    for norm, mats, n in (("norm1", ("w_in", "w_q", "w_k", "w_v"), cfg.d_model), ("gnorm", ("w_out",), cfg.d_inner),
                          ("norm2", ("w_gate", "w_up"), cfg.d_model)):
        c = np.exp2(r.integers(-6, 7, n)).astype(np.float32)
        _scale(scaled, "L0." + norm, c)
        for m in mats:
            _scale(scaled, "L0." + m, 1 / c)
    c = np.exp2(r.integers(-6, 7, cfg.d_ff)).astype(np.float32)
    _scale(scaled, "L0.w_up", c[:, None])
    _scale(scaled, "L0.w_down", 1 / c)
    worst = 0.0
    for got, ref in zip(_outputs(B, scaled, batch, k, tokens), _outputs(B, base, batch, k, tokens)):
        worst = max(worst, float(np.linalg.norm(got - ref) / np.linalg.norm(ref)))
    print(f"[columns-{batch}-{k}] {worst:.2e}", flush=True)
    assert worst < 1e-4
