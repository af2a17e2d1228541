"""Dense products of every kernel family against float64 (needs an MI355X): what reaches the next product is as accurate as float32
makes it, also for weights and activations of very different size.

A one- or two-block bf16 model is prefilled in one pass of batch x positions rows, which choose the kernels: 4..16 rows (activations
split per wavefront), 17..96 (per window, in either shape), more (split into planes beforehand, handed over or not), and the kernel of 9 rows and more
without LDS.  Compared are the raw convolution inputs, that is the input projection of each block, and the logits.  The reference
is the oracle with the library's own cached keys and values, so that no 16-bit rounding lies between the two.

Bound: 3e-6 of the compared vector's 2-norm.  Float32 leaves 7e-7 at most here (2^-24 per rounding, some hundred of them per sum, two
blocks); one 11-bit term alone, 2^-12 per value, would leave 1e-4."""
import numpy as np
import pytest

from oracle import hybrid_lm
from paper_2605_01106_amd import workloads as W

pytestmark = pytest.mark.gpu
BOUND = 3e-6

# rows of the pass, kernel flags by name
FAMILIES = [(2, 4, ()), (3, 5, ()), (4, 10, ()), (6, 16, ()), (10, 16, ()), (10, 16, ("HH_KF_NO_HANDOVER",)), (12, 50, ()),
            (3, 5, ("HH_KF_SKINNY_OFF", "HH_KF_MID_OFF")), (4, 15, ("HH_KF_MID_OFF",)), (4, 10, ("HH_KF_MID_OFF", "HH_KF_ROWS_LDS")),
            (4, 5, ("HH_KF_MID_WIDE",)), (3, 11, ("HH_KF_MID_WIDE",)), (4, 15, ("HH_KF_MID_WIDE",)), (7, 11, ("HH_KF_MID_WIDE",)), (6, 16, ("HH_KF_MID_WIDE",))]


def _model(layers=2, seed=11, d_model=264, d_ff=416):
    cfg = W.scaled_config("products", n_layers=layers, d_model=d_model, vocab=160, m_heads=16, m_head_dim=16, d_state=64, n_q_heads=4, n_kv_heads=2,
                          head_dim=32, d_ff=d_ff, w_dtype=W.BF16)
    wts = W.make_lively_weights(cfg, seed)
    for i in range(layers):           # an MLP that counts beside the two branches
        for name, factor in (("w_gate", 4), ("w_up", 4), ("w_down", 2)):
            _scale(wts, f"L{i}.{name}", factor)
    return cfg, wts


def _scale(wts, name, factor):
    put = wts.put_matrix if wts.values[name].ndim == 2 and not name.endswith("conv_w") else wts.put_vector
    put(name, (wts.values[name] * np.asarray(factor, np.float32)).astype(np.float32))


def _prefilled(wts, batch, tokens, flags=()):
    from paper_2605_01106_amd import binding as B

    bits = B.HH_KF_CANARIES
    for f in flags:
        bits |= getattr(B, f)
    prompts = W.make_prompts(wts.cfg.vocab, batch, [tokens] * batch, 6)
    ctx = B.Context(wts, batch, tokens + 20, 1, 8, kernel_flags=bits)
    ctx.hh_prefill(prompts, [tokens] * batch, 8)
    return ctx, prompts


def _reference(monkeypatch, wts, ctx, prompts, tokens):
    """float64 convolution windows [layer][batch] and logits [batch]"""
    cfg = wts.cfg
    lm = hybrid_lm.HybridLM(cfg, wts.values)
    windows, logits = [[] for _ in range(cfg.n_layers)], []
    for b in range(len(prompts)):
        kv = [ctx.hh_get_kv(layer, b, tokens) for layer in range(cfg.n_layers)]
        cached = iter([kv[layer][i][t] for t in range(tokens) for layer in range(cfg.n_layers) for i in range(2)])

        def stored(x, dtype):
            v = next(cached).astype(np.float64)
            assert np.abs(v - x).max() <= 2.0 ** -7 * np.abs(x).max()
            return v
        monkeypatch.setattr(hybrid_lm, "round_storage", stored)
        st = lm.new_state(tokens)
        for t in range(tokens):
            row = lm.step(st, int(prompts[b][t]))
        logits.append(row)
        for layer in range(cfg.n_layers):
            windows[layer].append(st.conv[layer])
    return [np.array(w) for w in windows], np.array(logits)


def _check(monkeypatch, wts, batch, tokens, flags, per_channel=False):
    ctx, prompts = _prefilled(wts, batch, tokens, flags)
    windows, logits = _reference(monkeypatch, wts, ctx, prompts, tokens)
    worst = {}
    for layer, ref in enumerate(windows):
        got = ctx.hh_get_state(layer)[1].astype(np.float64)
        axes = (0, 2) if per_channel else None
        err = np.sqrt(((got - ref) ** 2).sum(axis=axes) / (ref ** 2).sum(axis=axes))
        worst[f"conv{layer}"] = float(np.max(err))
    got = ctx.hh_get_logits(2).astype(np.float64)
    worst["logits"] = float(np.linalg.norm(got - logits) / np.linalg.norm(logits))
    assert ctx.hh_check_canaries() == 0
    print(f"[{batch}x{tokens} {' '.join(flags)}] " + " ".join(f"{k} {v:.1e}" for k, v in worst.items()), flush=True)
    assert max(worst.values()) < BOUND, worst


@pytest.mark.parametrize("batch,tokens,flags", FAMILIES)
def test_ordinary_weights(monkeypatch, batch, tokens, flags):
    _check(monkeypatch, _model()[1], batch, tokens, flags)


@pytest.mark.parametrize("batch,tokens,flags", FAMILIES)
def test_rows_of_very_different_size_in_one_tile(monkeypatch, batch, tokens, flags):
    """Rows of the input projection times 2^-26, the taps of their convolution times 2^26: each keeps its own accuracy."""
    cfg, wts = _model(layers=1)
    small = np.arange(cfg.conv_dim) % 3 == 1
    rows = np.ones(cfg.d_in_proj, np.float32)
    rows[cfg.d_inner:cfg.d_inner + cfg.conv_dim][small] = 2.0 ** -26
    _scale(wts, "L0.w_in", rows[:, None])
    _scale(wts, "L0.conv_w", np.where(small, np.float32(2.0 ** 26), np.float32(1))[:, None])
    _check(monkeypatch, wts, batch, tokens, flags, per_channel=True)


@pytest.mark.parametrize("batch,tokens,flags", FAMILIES)
def test_a_channel_that_outweighs_its_block(monkeypatch, batch, tokens, flags):
    """Every 40th norm weight times 2^22 and the columns that it meets divided by it: the same function, and the values beside it keep their
    accuracy."""
    cfg, wts = _model()
    for layer in range(cfg.n_layers):
        for norm, mats, n in (("norm1", ("w_in", "w_q", "w_k", "w_v"), cfg.d_model), ("gnorm", ("w_out",), cfg.d_inner), ("norm2", ("w_gate", "w_up"), cfg.d_model)):
            c = np.ones(n, np.float32)
            c[7::40] = 2.0 ** 22
            _scale(wts, f"L{layer}.{norm}", c)
            for name in mats:
                _scale(wts, f"L{layer}.{name}", 1 / c)
    _check(monkeypatch, wts, batch, tokens, flags)


@pytest.mark.parametrize("batch,tokens,flags", FAMILIES)
def test_mlp_columns_of_very_different_size(monkeypatch, batch, tokens, flags):
    """One channel of the second norm times 2^22 and its columns of gate and up divided by it, rows of up times 2^-12 to 2^12 and the columns
    of down divided by it: the same function, and the down projection's input keeps its accuracy."""
    cfg, wts = _model()
    r = np.random.default_rng(2)
    for layer in range(cfg.n_layers):
        c = np.ones(cfg.d_model, np.float32)
        c[77] = 2.0 ** 22
        _scale(wts, f"L{layer}.norm2", c)
        for name in ("w_gate", "w_up"):
            _scale(wts, f"L{layer}.{name}", 1 / c)
        c = np.exp2(r.integers(-12, 13, cfg.d_ff)).astype(np.float32)
        _scale(wts, f"L{layer}.w_up", c[:, None])
        _scale(wts, f"L{layer}.w_down", 1 / c)
    _check(monkeypatch, wts, batch, tokens, flags)


@pytest.mark.parametrize("batch,tokens,flags", FAMILIES)
def test_a_channel_that_outweighs_the_row(monkeypatch, batch, tokens, flags):
    """One channel of the residual stream 2^18 times the others, its norm weights 2^-18: what the MLP sees of a row is 2^-14 of what the norm
    allows, its result the square of that."""
    cfg, wts = _model()
    c = np.ones(cfg.d_model, np.float32)
    c[77] = 2.0 ** 18
    _scale(wts, "embed", c)
    _scale(wts, "final_norm", 1 / c)
    for layer in range(cfg.n_layers):
        for name in ("norm1", "norm2"):
            _scale(wts, f"L{layer}.{name}", 1 / c)
        for name in ("w_gate", "w_up"):
            _scale(wts, f"L{layer}.{name}", 2.0 ** 14)
    _check(monkeypatch, wts, batch, tokens, flags)


# widths at which gate/up and down of 8 rows take different kernels: the vector unit for the one, the matrix cores for the other
@pytest.mark.parametrize("d_model,d_ff", [(2592, 416), (264, 5128), (2592, 5128)])
def test_mlp_products_of_different_kernels(monkeypatch, d_model, d_ff):
    _check(monkeypatch, _model(d_model=d_model, d_ff=d_ff)[1], 2, 4, ())


@pytest.mark.parametrize("batch,tokens,flags", FAMILIES)
def test_an_infinite_weight_stays_in_its_row(batch, tokens, flags):
    """The rows beside one with an infinite weight: the same bits as without it."""
    cfg, wts = _model(layers=1)
    ctx, _ = _prefilled(wts, batch, tokens, flags)
    ref = ctx.hh_get_state(0)[1]
    channel = 37
    w = wts.values["L0.w_in"].copy()
    w[cfg.d_inner + channel, 5] = np.inf
    wts.put_matrix("L0.w_in", w)
    ctx, _ = _prefilled(wts, batch, tokens, flags)
    got = ctx.hh_get_state(0)[1]
    assert not np.isfinite(got[:, channel]).any()
    others = np.arange(cfg.conv_dim) != channel
    assert np.array_equal(got[:, others], ref[:, others])
