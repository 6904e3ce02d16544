"""Products whose K ranges meet in memory: tiles over ranges of K, ragged in rows and columns, and the kernel that sums the
ranges eight columns a thread, where the last of its blocks is partly empty; through the MLP phase of a layer and against the
CPU oracle.  (test_product_routes.py checks that every product named here is cut as said.)"""
import pytest
import torch

import workloads as wl
from oracle import layer_math as lm

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2503_06433_amd as ss
    from paper_2503_06433_amd.harness import make_context, to_device, to_f64, empty_like_acts, parity, pp_desc


@pytest.mark.parametrize("dtype,T,hidden,ffn", [
    (wl.BF16, 261, 12288, 1056),       # tiles of the gate / up product in four ranges: 261 x 132 pieces, 134.6 blocks
    (wl.F16, 97, 1096, 12800),         # register-staged kernel, down in eight ranges, with and without a residual: 97 x 137 pieces, 51.9 blocks
    (wl.BF16, 601, 4160, 11008),       # persistent kernel, down in four ranges: 601 x 520 pieces, 1220.8 blocks
    (wl.F16, 700, 4112, 8192),         # ... in four, the last tiles' rows and columns cut short
    (wl.BF16, 81, 8192, 640),          # tiles of the gate / up product in eight ranges
    (wl.F16, 141, 1096, 12288),        # ... of the down projection in eight, the last ones wider than what is left of the output
    (wl.BF16, 333, 2088, 8192),        # ... in four
    (wl.BF16, 120, 5120, 1056),        # ... of the gate / up product in eight ranges of ten slices
])
def test_summed_ranges_match_oracle(dtype, T, hidden, ffn):
    cfg = wl.ModelCfg(hidden=hidden, n_q_heads=1, n_kv_heads=1, head_dim=64, ffn=ffn, n_layers=1, dtype=dtype)
    vals, raws = wl.make_layer_weights(cfg, 971)
    ctx = make_context(cfg, pages=4, max_seq_len=64)
    d = pp_desc(cfg)
    ctx.load_layer(d, 0, raws)
    xv, xr = wl.make_activations((T, hidden), 972, dtype)
    ref = lm.mlp_block(cfg, vals, xv, 1, 0)
    for phase, add in ((ss.SS_MLP, xv), (ss.SS_MLP | ss.SS_NO_RESIDUAL, 0.0)):
        out = empty_like_acts(T + 1, hidden, dtype)
        out.fill_(7.0)
        ctx.layer_prefill(d, 0, phase, list(range(T)), [1] * T, [0] * T, to_device(xr, dtype), out)
        torch.cuda.synchronize()
        got = to_f64(out, dtype)
        assert (got[T] == 7.0).all()
        parity(got[:T], ref + add, dtype, "summed ranges, %d rows, hidden %d, ffn %d" % (T, hidden, ffn))
    ctx.destroy()
