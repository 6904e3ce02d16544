"""A decode batch that lists a sequence at several of its positions (tokens in the cache already, taken again): every entry
attends to the new keys and values of the others in front of it, as the same tokens give one call after the other."""
import numpy as np
import pytest
import torch

import workloads as wl

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2503_06433_amd as ss
    from paper_2503_06433_amd.harness import make_context, pp_desc, to_f64, torch_dtype, empty_like_acts, parity

IDS, AT, LENS = [5, 9, 5, 5, 5], [48, 33, 40, 47, 41], {5: 60, 9: 33}       # sequence 9 brings an ordinary new token


@pytest.mark.parametrize("dtype,nq,nkv,d", [(wl.BF16, 4, 2, 128), (wl.F16, 2, 2, 128), (wl.BF16, 20, 1, 128), (wl.F32, 4, 2, 64)])
def test_positions_of_one_sequence_see_each_other(dtype, nq, nkv, d):
    cfg = wl.ModelCfg(hidden=128, n_q_heads=nq, n_kv_heads=nkv, head_dim=d, ffn=64, n_layers=1, dtype=dtype)
    _, raws = wl.make_layer_weights(cfg, 981)
    gen = torch.Generator(device="cuda").manual_seed(982)
    fill = lambda *s: torch.empty(s, device="cuda", dtype=torch_dtype(dtype)).normal_(0, 1, generator=gen)
    staging, x, desc = fill(sum(LENS.values()) * 2 * nkv * d), fill(len(IDS), cfg.hidden), pp_desc(cfg)
    together, apart = [list(range(len(IDS)))], [[i] for i in np.argsort(AT)]
    outs, caches = [], []
    for calls in (together, together + together, apart):                 # the second with the metadata of the first
        ctx = make_context(cfg, pages=16, max_seq_len=128)
        ctx.load_layer(desc, 0, raws)
        ctx.kv_import_dev(desc, list(LENS), list(LENS.values()), staging)
        out = empty_like_acts(len(IDS), cfg.hidden, dtype)
        for rows in calls:
            y = empty_like_acts(len(rows), cfg.hidden, dtype)
            ctx.layer_decode(desc, 0, ss.SS_ATTN | ss.SS_NO_RESIDUAL, [IDS[i] for i in rows], [AT[i] for i in rows], x[rows].contiguous(), y)
            out[rows] = y
        torch.cuda.synchronize()
        outs.append(to_f64(out, dtype))
        caches.append([ctx.kv_read(desc, i, 0, nkv) for i in LENS])
        ctx.destroy()
    for i in range(2):
        parity(outs[i], outs[2], dtype, "positions of one sequence in one batch, %d heads over %d of %d" % (nq, nkv, d))
        for a, b in zip(caches[i], caches[2]):
            a, b = (a, b) if dtype == wl.F32 else (a.astype(np.int32), b.astype(np.int32))
            assert np.array_equal(a, b) if dtype == wl.BF16 else np.abs(a - b).max() <= (1 if dtype == wl.F16 else 1e-5)
