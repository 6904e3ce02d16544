"""Decode attention rotates the new token and writes its page by itself; a prefill call of one token does it in a kernel of
its own.  Both leave the same bits in the cache and agree on the output, for cached lengths around page edges, page pairs and the
lengths at which a sequence gets a second and third work item."""
import numpy as np
import pytest
import torch

import workloads as wl

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2503_06433_amd as ss
    from paper_2503_06433_amd.harness import make_context, pp_desc, to_f64, torch_dtype, empty_like_acts, parity

LENS = [0, 1, 14, 15, 16, 17, 31, 32, 33, 47, 48, 63, 64, 255, 256, 257, 300, 511, 512, 1000]


@pytest.mark.parametrize("dtype,nq,nkv,d,lens", [
    (wl.BF16, 4, 4, 128, LENS),
    (wl.BF16, 16, 1, 128, LENS),       # all sixteen query columns in use
    (wl.F16, 6, 2, 128, LENS),
    (wl.F16, 20, 1, 128, LENS),        # from here on the plain kernel: more heads than columns, other widths, fp32
    (wl.BF16, 4, 2, 64, LENS),
    (wl.F32, 4, 2, 64, LENS),
    (wl.F32, 4, 1, 128, LENS),
    (wl.F32, 32, 2, 64, LENS),         # so many heads that a kernel of its own rotates and writes for the plain one
    (wl.BF16, 64, 4, 64, LENS),
    (wl.F16, 64, 1, 128, LENS),
    (wl.F16, 8, 8, 64, LENS),
    (wl.F16, 16, 16, 128, LENS),       # two thousand key values a token: some land on a tie
    (wl.F32, 80, 2, 64, LENS[:10]),      # no sequence of more than four pages
    (wl.F32, 8, 2, 128, LENS[:10]),
    (wl.F16, 17, 17, 128, [0] + [1 + i % 37 for i in range(255)]),
    (wl.BF16, 16, 16, 128, [0] + [1 + i % 40 for i in range(255)]),      # so many waves of few pages that a kernel of its own does it for both
])
def test_decode_leaves_the_cache_of_a_one_token_prefill(dtype, nq, nkv, d, lens):
    cfg = wl.ModelCfg(hidden=128, n_q_heads=nq, n_kv_heads=nkv, head_dim=d, ffn=64, n_layers=1, dtype=dtype)
    _, raws = wl.make_layer_weights(cfg, 951)
    gen = torch.Generator(device="cuda").manual_seed(952)
    fill = lambda *s: torch.empty(s, device="cuda", dtype=torch_dtype(dtype)).normal_(0, 1, generator=gen)
    staging, x = fill(sum(lens) * 2 * nkv * d), fill(len(lens), cfg.hidden)
    ids, desc, outs, caches = list(range(len(lens))), pp_desc(cfg), [], []
    for decode in (True, False):
        ctx = make_context(cfg, pages=sum(n // 16 + 1 for n in lens), max_seq_len=1024)
        ctx.load_layer(desc, 0, raws)
        ctx.kv_import_dev(desc, ids[1:], lens[1:], staging)
        out = empty_like_acts(len(lens), cfg.hidden, dtype)
        if decode:
            ctx.layer_decode(desc, 0, ss.SS_ATTN | ss.SS_NO_RESIDUAL, ids, lens, x, out)
        else:
            ctx.layer_prefill(desc, 0, ss.SS_ATTN | ss.SS_NO_RESIDUAL, ids, [1] * len(ids), lens, x, out)
        torch.cuda.synchronize()
        outs.append(to_f64(out, dtype))
        caches.append([ctx.kv_read(desc, i, 0, nkv) for i in ids])
        ctx.destroy()
    for i, n in enumerate(lens):
        assert caches[0][i].shape[2] == n + 1
        a, b = (c[i] if dtype == wl.F32 else c[i].astype(np.int32) for c in caches)
        assert np.array_equal(a, b), "%d cached tokens" % n
    parity(outs[0], outs[1], dtype, "decode against a one-token prefill, %d heads over %d of %d" % (nq, nkv, d))
