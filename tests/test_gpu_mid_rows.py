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


# (rows, hidden, ffn) whose gate / up product (SwiGLU) or down projection takes the tile at this place of the list: tiles of
# one, eleven (fewer and more than the ring has stages) or ten slices, output edges inside the tiles.
GATE_UP_TILES = {
    0: (65, 640, 64), 1: (4501, 640, 96), 2: (65, 704, 64), 3: (1001, 704, 768), 4: (4501, 640, 64), 5: (4501, 704, 128),
    6: (1201, 704, 1216), 7: (5001, 704, 160), 8: (5001, 704, 224), 9: (5001, 704, 320), 10: (4501, 704, 672), 11: (3001, 704, 512),
    12: (5001, 704, 416), 13: (5001, 704, 448), 14: (5001, 704, 800), 15: (5001, 704, 608), 16: (5001, 704, 896), 17: (5001, 704, 992),
}
DOWN_TILES = {
    0: (65, 64, 640), 1: (4501, 192, 640), 2: (65, 64, 704), 3: (1001, 1536, 704), 4: (4501, 128, 640), 5: (4501, 256, 704),
    6: (1201, 2432, 704), 7: (5001, 320, 704), 8: (5001, 448, 704), 9: (5001, 640, 704), 10: (4501, 1344, 704), 11: (3001, 1024, 704),
    12: (5001, 832, 704), 13: (5001, 896, 704), 14: (5001, 1600, 704), 15: (5001, 1216, 704), 16: (5001, 1792, 704), 17: (5001, 1984, 704),
}


@pytest.mark.parametrize("product,tile", [("gate/up", t) for t in GATE_UP_TILES] + [("down", t) for t in DOWN_TILES])
def test_every_tile_matches_oracle(product, tile):
    T, hidden, ffn = (GATE_UP_TILES if product == "gate/up" else DOWN_TILES)[tile]
    dtype = wl.F16 if tile % 3 == 2 else wl.BF16
    cfg = wl.ModelCfg(hidden=hidden, n_q_heads=1, n_kv_heads=1, head_dim=64, ffn=ffn, n_layers=1, dtype=dtype)
    vals, raws = wl.make_layer_weights(cfg, 981)
    ctx = make_context(cfg, pages=4, max_seq_len=64)
    d = pp_desc(cfg)
    ctx.load_layer(d, 0, raws)
    xv, xr = wl.make_activations((T, hidden), 982, dtype)
    # rows are independent: the first and last ones, both sides of every tile edge, and some in between
    edges = {e + o for bm in (64, 96) for e in range(0, T, bm) for o in (-1, 0)} | set(range(7, T, 61)) | set(range(max(0, T - 70), T))
    rows = np.array(sorted(r for r in edges if r >= 0))
    ref = lm.mlp_block(cfg, vals, xv[rows], 1, 0)
    for phase, add in ((ss.SS_MLP, xv[rows]), (ss.SS_MLP | ss.SS_NO_RESIDUAL, 0.0)):
        out = empty_like_acts(T + 1, hidden, dtype)
        out.fill_(7.0)
        ctx.layer_prefill(d, 0, phase, list(range(T)), [1] * T, [0] * T, to_device(xr, dtype), out)
        torch.cuda.synchronize()
        got = to_f64(out, dtype)
        assert (got[T] == 7.0).all() and np.isfinite(got).all()
        parity(got[rows], ref + add, dtype, "tile %d, %s of %d rows, hidden %d, ffn %d" % (tile, product, T, hidden, ffn))
    ctx.destroy()
