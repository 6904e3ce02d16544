"""One infinite value in the cache (an activation that overflowed the storage type) through decode attention: its
element of the head is infinite, everything else is as it was, whatever the number of partial results that are merged."""
import pytest
import torch

import workloads as wl

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2503_06433_amd as ss
    from paper_2503_06433_amd.harness import make_context, pp_desc, to_f64, torch_dtype, empty_like_acts

LENS = [20, 300, 700, 1000, 1200]         # one to five work items of 16 pages; the page of the value is never a repeated one


@pytest.mark.parametrize("dtype", [wl.BF16, wl.F16])
def test_infinite_value_stays_infinite_in_the_merged_result(dtype):
    cfg = wl.ModelCfg(hidden=256, n_q_heads=2, n_kv_heads=2, head_dim=128, ffn=64, n_layers=1, dtype=dtype)
    _, raws = wl.make_layer_weights(cfg, 931)
    ctx = make_context(cfg, pages=sum(n // 16 + 2 for n in LENS), max_seq_len=1300)
    d = pp_desc(cfg)
    ctx.load_layer(d, 0, raws)
    gen = torch.Generator(device="cuda").manual_seed(932)
    runs = [torch.empty((2, 2, n, 128), device="cuda", dtype=torch_dtype(dtype)).normal_(0, 1, generator=gen) for n in LENS]
    x = torch.empty((len(LENS), cfg.hidden), device="cuda", dtype=torch_dtype(dtype)).normal_(0, 1, generator=gen)
    ids, out = list(range(len(LENS))), empty_like_acts(len(LENS), cfg.hidden, dtype)
    wo = to_f64(torch.from_numpy(raws["wo"].view("int16")).view(torch_dtype(dtype)), dtype)
    for sign in (1.0, -1.0):
        for r in runs:
            r[1, 0, 2, 7] = sign * float("inf")           # V of head 0, token 2, element 7
        ctx.kv_import_dev(d, ids, LENS, torch.cat([r.reshape(-1) for r in runs]))
        ctx.layer_decode(d, 0, ss.SS_ATTN | ss.SS_NO_RESIDUAL, ids, LENS, x, out)
        torch.cuda.synchronize()
        got = to_f64(out, dtype)
        assert (wo[7] != 0).all()
        for i, n in enumerate(LENS):
            assert (got[i] == sign * wo[7] * float("inf")).all(), "%d cached tokens" % n
        ctx.kv_free(d, ids)
    ctx.destroy()
