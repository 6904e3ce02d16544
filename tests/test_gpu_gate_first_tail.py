"""SwiGLU of layers whose gate rows come first (hidden size no multiple of 64) far down its left tail, where
1 + exp(-g) is above 2^126 and its reciprocal below the smallest normal number: the quotient itself is a normal bf16."""
import numpy as np
import pytest
import torch

import workloads as wl

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2503_06433_amd as ss
    from paper_2503_06433_amd.harness import make_context, pp_desc, to_f64, empty_like_acts


@pytest.mark.parametrize("T", [1, 16, 64, 65])
def test_left_tail_of_swiglu_keeps_its_precision(T):
    cfg = wl.ModelCfg(hidden=72, n_q_heads=1, n_kv_heads=1, head_dim=64, ffn=64, n_layers=1, dtype=wl.BF16)
    _, raws = wl.make_layer_weights(cfg, 961)
    gate = wl.bf16_to_f32(wl.bf16_bits(np.array([-88.0 / 72], dtype=np.float32)))[0]
    for name, v in (("g1", 1.0), ("g2", 1.0), ("wg", gate), ("wu", 0.5), ("wd", 1.0)):
        raws[name] = wl.bf16_bits(np.full(raws[name].shape, v, dtype=np.float32))
    ctx = make_context(cfg, pages=T + 2, max_seq_len=32)
    d = pp_desc(cfg)
    ctx.load_layer(d, 0, raws)
    x, out = torch.ones((T, 72), device="cuda", dtype=torch.bfloat16), empty_like_acts(T, 72, wl.BF16)
    ctx.layer_prefill(d, 0, ss.SS_MLP | ss.SS_NO_RESIDUAL, list(range(T)), [1] * T, [0] * T, x, out)
    torch.cuda.synchronize()
    g = 72 * float(gate) / np.sqrt(1.0 + cfg.rms_eps)
    ref = 64 * g / (1.0 + np.exp(-g)) * 36.0 / np.sqrt(1.0 + cfg.rms_eps)
    got = to_f64(out, wl.BF16)
    # Up to 64 rows the gate stays in fp32: its sums are off by at most 72 * 2^-24 of it, which changes exp(-g) by 88 times
    # that, and the activation and the result are rounded to 8 bits.  Above, gate and up are stored in 8 bits in between:
    # half a unit of 0.5 at 88, and one more rounding.
    bound = 88 * 72 * 2.0 ** -24 + 2 * 2.0 ** -8 if T <= 64 else np.expm1(0.25) + 3 * 2.0 ** -8
    assert np.abs(got / ref - 1).max() <= bound, (got.min(), got.max(), ref)
    ctx.destroy()
