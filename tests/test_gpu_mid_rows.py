"""Products of 65 to some hundred token rows (the kernel that picks its output tile by shape and splits K between groups of
waves of a block), through the MLP phase of a layer and against the CPU oracle: row counts around the tile edges, contractions
of fewer slices than the ring has stages, of an odd number of slices, and longer ones, output widths that end inside a tile."""
import numpy as np
import pytest
import torch

import workloads as wl
from oracle import layer_math as lm

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2503_06433_amd as ss
    from paper_2503_06433_amd.harness import make_context, to_device, to_f64, empty_like_acts, parity, pp_desc


@pytest.mark.parametrize("dtype,hidden,ffn", [
    (wl.BF16, 64, 64),         # one slice, one tile
    (wl.BF16, 192, 1088),      # three and seventeen slices (no stages of two slices), gate / up tiles that end inside
    (wl.F16, 512, 2304),
    (wl.F16, 192, 12800),      # up to 128 rows the down projection is cut along its 200 slices
    (wl.BF16, 1344, 8192),     # tiles of 128 weight rows and more for the gate / up product
])
def test_mlp_of_middling_row_counts_matches_oracle(dtype, hidden, ffn):
    cfg = wl.ModelCfg(hidden=hidden, n_q_heads=1, n_kv_heads=1, head_dim=64, ffn=ffn, n_layers=1, dtype=dtype)
    vals, raws = wl.make_layer_weights(cfg, 911)
    ctx = make_context(cfg, pages=400, max_seq_len=64)
    d = pp_desc(cfg)
    ctx.load_layer(d, 0, raws)
    for T in (65, 96, 97, 128, 129, 192, 193, 257, 333):
        xv, xr = wl.make_activations((T, hidden), 912 + T, dtype)
        for phase, with_res in ((ss.SS_MLP, True), (ss.SS_MLP | ss.SS_NO_RESIDUAL, False)):
            out = empty_like_acts(T + 1, hidden, dtype)
            out.fill_(7.0)
            ctx.layer_prefill(d, 0, phase, list(range(T)), [1] * T, [0] * T, to_device(xr, dtype), out)
            torch.cuda.synchronize()
            got = to_f64(out, dtype)
            assert (got[T] == 7.0).all()                      # nothing is written behind the last row
            ref = lm.mlp_block(cfg, vals, xv, 1, 0)
            parity(got[:T], ref + xv if with_res else ref, dtype, "MLP of %d rows, hidden %d, ffn %d" % (T, hidden, ffn))
    ctx.destroy()
