"""Products of few token rows (the kernel that loads both operands straight into matrix-instruction registers, works
out the RMSNorm factor of its rows itself and applies SwiGLU and residual to finished sums), through the MLP phase of
a layer and against the CPU oracle: row counts around every tile edge, output widths that select one, two and three
weight tiles per block, contractions that end inside a 128-byte chunk, both layouts of the gate / up rows."""
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
    (wl.BF16, 128, 1024),      # one tile per block
    (wl.BF16, 192, 3104),      # two; the down projection's contraction ends inside a chunk
    (wl.F16, 128, 5152),       # three
    (wl.F16, 128, 8224),       # three up to 16 rows, and a long contraction for one wave's share
    (wl.BF16, 128, 12800),     # gate / up so wide that more than 16 rows take the tile kernel, a contraction so long that more
                               # than 32 take split K in front of it
    (wl.BF16, 2112, 4128),     # contractions of 2048 and more: three tiles; down sixteen waves that share 65 chunks, the last cut
    (wl.F16, 2048, 2752),      # sixteen waves of two tiles from 9 rows on
    (wl.BF16, 2080, 7200),     # four tiles; a cut chunk behind whole ones that are no multiple of those on their way
    (wl.BF16, 4160, 8200),     # down up to 8 rows two tiles
    (wl.BF16, 200, 72),        # hidden no multiple of 64: gate rows first, up rows behind; chunks cut on both sides
    (wl.F32, 256, 688),
    (wl.F32, 36, 4100),        # fp32 with three tiles per block and a contraction of little more than one chunk
])
def test_mlp_of_few_rows_matches_oracle(dtype, hidden, ffn):
    cfg = wl.ModelCfg(hidden=hidden, n_q_heads=1, n_kv_heads=1, head_dim=64, ffn=ffn, n_layers=1, dtype=dtype)
    vals, raws = wl.make_layer_weights(cfg, 901)
    ctx = make_context(cfg, pages=80, max_seq_len=64)
    d = pp_desc(cfg)
    ctx.load_layer(d, 0, raws)
    for T in (1, 8, 9, 16, 17, 32, 33, 48, 49, 64, 65):
        xv, xr = wl.make_activations((T, hidden), 902 + T, dtype)
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
