"""One query per sequence through the plain attention kernel (fp32, head dimension 64, more than 16 query heads per kv
head) against the CPU oracle: cached lengths around page edges and around the point where each of the four waves of a
block has its first and second page."""
import numpy as np
import pytest
import torch

import workloads as wl
from oracle import layer_math as lm

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2503_06433_amd as ss
    from paper_2503_06433_amd.harness import make_context, to_device, to_f64, empty_like_acts, parity, pp_desc

LENS = [1, 15, 16, 17, 31, 47, 48, 63, 64, 65, 79, 127, 128, 200]


@pytest.mark.parametrize("dtype,nq,nkv,d", [
    (wl.F32, 4, 4, 64),
    (wl.F32, 4, 1, 128),
    (wl.BF16, 4, 2, 64),
    (wl.F16, 20, 1, 128),        # a group of more heads than the matrix-instruction kernel has columns
])
def test_one_query_per_sequence_matches_oracle(dtype, nq, nkv, d):
    cfg = wl.ModelCfg(hidden=128, n_q_heads=nq, n_kv_heads=nkv, head_dim=d, ffn=64, n_layers=1, dtype=dtype)
    vals, raws = wl.make_layer_weights(cfg, 911)
    ctx = make_context(cfg, pages=sum(-(-(n + 1) // 16) for n in LENS) + 4, max_seq_len=256)
    desc = pp_desc(cfg)
    ctx.load_layer(desc, 0, raws)
    n, ids = len(LENS), list(range(len(LENS)))
    rk = {wl.F32: None, wl.BF16: lambda a: wl.bf16_to_f32(wl.bf16_bits(a.astype(np.float32))).astype(np.float64),
          wl.F16: lambda a: a.astype(np.float16).astype(np.float64)}[dtype]
    cache = lm.KVCache(cfg)
    xv, xr = wl.make_activations((sum(LENS), cfg.hidden), 912, dtype)
    out = empty_like_acts(sum(LENS), cfg.hidden, dtype)
    ctx.layer_prefill(desc, 0, ss.SS_ATTN, ids, LENS, [0] * n, to_device(xr, dtype), out)
    lm.attn_block(cfg, vals, xv, [(i, m, 0) for i, m in zip(ids, LENS)], cache, 0, 1, 0, rk)
    dv, dr = wl.make_activations((n, cfg.hidden), 913, dtype)
    got = empty_like_acts(n, cfg.hidden, dtype)
    ctx.layer_decode(desc, 0, ss.SS_ATTN | ss.SS_NO_RESIDUAL, ids, LENS, to_device(dr, dtype), got)
    torch.cuda.synchronize()
    ref = lm.attn_block(cfg, vals, dv, [(i, 1, m) for i, m in zip(ids, LENS)], cache, 0, 1, 0, rk)
    parity(to_f64(got, dtype), ref, dtype, "one query per sequence, %d heads over %d of %d" % (nq, nkv, d))
    ctx.destroy()
