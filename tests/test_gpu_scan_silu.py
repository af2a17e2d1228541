"""The SiLU of the scans against float64 (needs an MI355X), read from the state behind one position: taps of 0 and 1, B = silu(64) = 64 and a step
size of 32 leave S = 2048 silu(x) exactly, and the convolution window holds x.

Bound: the division rounds once.  Of the values below, |x| < 2, the form with one rounding is off by 4.3e-8 to 4.5e-8 rms, one that rounds the
reciprocal as well by 5.0e-8 to 5.2e-8."""
import numpy as np
import pytest

from paper_2605_01106_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d_state", [16, 64, 128])
@pytest.mark.parametrize("flag", ["", "HH_KF_SSM_GENERAL", "HH_KF_SSM_SCALAR_CONV"])
def test_one_rounding(flag, d_state):
    from paper_2605_01106_amd import binding as B

    cfg = W.scaled_config("silu", n_layers=1, d_model=64, vocab=160, m_heads=16, m_head_dim=64, d_state=d_state, n_q_heads=2, n_kv_heads=1, head_dim=32,
                          d_ff=96, w_dtype=W.F32)
    wts, batch, di = W.make_lively_weights(cfg, 5), 64, cfg.d_inner
    conv_w, conv_b = np.zeros((cfg.conv_dim, 4), np.float32), np.full(cfg.conv_dim, 64, np.float32)
    conv_w[:di, 3], conv_b[:di] = 1, 0
    w_in = wts.values["L0.w_in"].copy()
    w_in[di + cfg.conv_dim:] = 0
    for name, v in (("conv_b", conv_b), ("dt_bias", np.full(cfg.m_heads, 32, np.float32))):
        wts.put_vector("L0." + name, v)
    wts.put_vector("L0.conv_w", conv_w)
    wts.put_matrix("L0.w_in", w_in)
    ctx = B.Context(wts, batch, 40, 1, 8, kernel_flags=(getattr(B, flag) if flag else 0) | B.HH_KF_CANARIES)
    ctx.hh_prefill(W.make_prompts(cfg.vocab, batch, 1, 3), [1] * batch, 8)
    state, window = ctx.hh_get_state(0)
    x = window[:, :di, 2].astype(np.float64)
    got = state.reshape(batch, di, d_state)
    assert (got == got[:, :, :1]).all()
    ref = 2048 * x / (1 + np.exp(-x))
    near = np.abs(x) < 2
    err = (got[:, :, 0] - ref)[near] / ref[near]
    rms = float(np.sqrt((err ** 2).mean()))
    print(f"[silu {flag} {d_state}] {near.sum()} values rms {rms:.3e}", flush=True)
    assert near.sum() > 20000 and rms < 4.75e-8
