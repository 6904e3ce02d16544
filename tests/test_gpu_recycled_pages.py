"""Pages whose last owner left values that are not finite behind the tokens of the present one: decode, whole prompts, a
prompt's second chunk and one-token rows of a prefill call give the same bits as with pages that were never used."""
import pytest
import torch

import workloads as wl

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2503_06433_amd as ss
    from paper_2503_06433_amd.harness import make_context, pp_desc, torch_dtype, empty_like_acts

OLD = [160, 400, 700]                    # first owners, whole pages
#        (new tokens, cached before them) of the three sequences that get the pages
CALLS = [("decode", [1, 1, 1], [16, 130, 320]),        # behind one and twenty whole pages, inside one that the import has filled up
         ("prefill", [5, 33, 64], [0, 0, 0]),          # per-wave loads
         ("prefill", [1, 1, 1], [2, 35, 300]),
         ("prefill", [70, 333, 600], [0, 0, 0]),       # tiles of 64 tokens in LDS; blocks of 256 queries that end inside a tile
         ("prefill", [100, 7, 257], [37, 64, 130])]


@pytest.mark.parametrize("dtype,nq,nkv,d", [(wl.BF16, 4, 2, 128), (wl.F16, 2, 2, 128), (wl.F16, 20, 1, 128), (wl.BF16, 4, 2, 64),
                                            (wl.F32, 4, 2, 64), (wl.F32, 2, 1, 128)])
def test_what_an_earlier_owner_left_is_not_seen(dtype, nq, nkv, d):
    cfg = wl.ModelCfg(hidden=128, n_q_heads=nq, n_kv_heads=nkv, head_dim=d, ffn=64, n_layers=1, dtype=dtype)
    _, raws = wl.make_layer_weights(cfg, 921)
    gen = torch.Generator(device="cuda").manual_seed(922)
    fill = lambda *s: torch.empty(s, device="cuda", dtype=torch_dtype(dtype)).normal_(0, 1, generator=gen)
    desc, ids = pp_desc(cfg), [11, 12, 13]
    for kind, new, before in CALLS:
        x, cached = fill(sum(new), cfg.hidden), fill(max(1, sum(before)) * 2 * nkv * d)
        outs = []
        for bad in (None, float("inf"), float("nan")):
            ctx = make_context(cfg, pages=sum(OLD) // 16 + 3, max_seq_len=1024)
            ctx.load_layer(desc, 0, raws)
            if bad is not None:
                ctx.kv_import_dev(desc, [1, 2, 3], OLD, torch.full((sum(OLD) * 2 * nkv * d,), bad, device="cuda", dtype=torch_dtype(dtype)))
                ctx.kv_free(desc, [1, 2, 3])
            old = [i for i, n in zip(ids, before) if n]
            if old:
                ctx.kv_import_dev(desc, old, [n for n in before if n], cached)
            out = empty_like_acts(sum(new), cfg.hidden, dtype)
            if kind == "decode":
                ctx.layer_decode(desc, 0, ss.SS_ATTN | ss.SS_NO_RESIDUAL, ids, before, x, out)
            else:
                ctx.layer_prefill(desc, 0, ss.SS_ATTN | ss.SS_NO_RESIDUAL, ids, new, before, x, out)
            torch.cuda.synchronize()
            outs.append(out.float().cpu())
            ctx.destroy()
        assert torch.isfinite(outs[0]).all()
        for o in outs[1:]:
            assert torch.equal(o, outs[0]), "%s %s behind %s" % (kind, new, before)


@pytest.mark.parametrize("dtype", [wl.BF16, wl.F16])
def test_many_short_sequences_on_recycled_pages(dtype):
    """4096 waves of the matrix-core kernel and a page or two each: the new tokens are rotated and written in front of it."""
    cfg = wl.ModelCfg(hidden=128, n_q_heads=16, n_kv_heads=16, head_dim=128, ffn=64, n_layers=1, dtype=dtype)
    _, raws = wl.make_layer_weights(cfg, 923)
    gen = torch.Generator(device="cuda").manual_seed(924)
    fill = lambda *s: torch.empty(s, device="cuda", dtype=torch_dtype(dtype)).normal_(0, 1, generator=gen)
    desc, ids = pp_desc(cfg), list(range(256))
    lens = [(16, 1, 30, 32)[i % 4] for i in ids]          # a new page, two inside one, another new page
    x, cached, outs = fill(256, cfg.hidden), fill(sum(lens) * 2 * 16 * 128), []
    for bad in (None, float("inf"), float("nan")):
        ctx = make_context(cfg, pages=256 * 3, max_seq_len=64)
        ctx.load_layer(desc, 0, raws)
        if bad is not None:
            old = [1000 + i for i in ids]
            ctx.kv_import_dev(desc, old, [48] * 256, torch.full((256 * 48 * 2 * 16 * 128,), bad, device="cuda", dtype=torch_dtype(dtype)))
            ctx.kv_free(desc, old)
        ctx.kv_import_dev(desc, ids, lens, cached)
        out = empty_like_acts(256, cfg.hidden, dtype)
        ctx.layer_decode(desc, 0, ss.SS_ATTN | ss.SS_NO_RESIDUAL, ids, lens, x, out)
        torch.cuda.synchronize()
        outs.append(out.float().cpu())
        ctx.destroy()
    assert torch.isfinite(outs[0]).all()
    assert torch.equal(outs[1], outs[0]) and torch.equal(outs[2], outs[0])
