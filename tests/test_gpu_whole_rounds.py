"""Products of a little more than a whole number of rounds of 256 x 256 tiles: the persistent kernel takes the columns of its
whole rounds, the tile kernel the rest.  Through the MLP phase of a layer and against the CPU oracle, with every epilogue of a
layer, ragged in rows and columns, an odd number of slices."""
import numpy as np
import pytest
import torch

import workloads as wl
from oracle import layer_math as lm

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2503_06433_amd as ss
    from paper_2503_06433_amd.harness import make_context, to_device, to_f64, empty_like_acts, parity, pp_desc


@pytest.mark.parametrize("dtype,T,hidden,ffn", [
    (wl.BF16, 4123, 4160, 2112),       # 17 x 17 tiles in both products, 15 columns of them in the round; 65 and 33 slices
    (wl.F16, 4355, 3904, 2048),        # 18 x 16 tiles, 14 columns; the rest of the down projection ends inside a tile
])
def test_cut_products_match_oracle(dtype, T, hidden, ffn):
    cfg = wl.ModelCfg(hidden=hidden, n_q_heads=1, n_kv_heads=1, head_dim=64, ffn=ffn, n_layers=1, dtype=dtype)
    vals, raws = wl.make_layer_weights(cfg, 961)
    ctx = make_context(cfg, pages=4, max_seq_len=64)
    d = pp_desc(cfg)
    ctx.load_layer(d, 0, raws)
    xv, xr = wl.make_activations((T, hidden), 962, dtype)
    # rows are independent: the first and last ones, both sides of the tile edges, and some in between
    edges = {e + o for e in range(0, T, 256) for o in (-1, 0)} | set(range(7, T, 61)) | set(range(T - 40, T))
    rows = np.array(sorted(r for r in edges if r >= 0))
    ref = lm.mlp_block(cfg, vals, xv[rows], 1, 0)
    for phase, add in ((ss.SS_MLP, xv[rows]), (ss.SS_MLP | ss.SS_NO_RESIDUAL, 0.0)):
        out = empty_like_acts(T + 1, hidden, dtype)
        out.fill_(7.0)
        ctx.layer_prefill(d, 0, phase, list(range(T)), [1] * T, [0] * T, to_device(xr, dtype), out)
        torch.cuda.synchronize()
        got = to_f64(out, dtype)
        assert (got[T] == 7.0).all() and np.isfinite(got).all()
        parity(got[rows], ref + add, dtype, "cut products, %d rows, hidden %d, ffn %d" % (T, hidden, ffn))
    ctx.destroy()
