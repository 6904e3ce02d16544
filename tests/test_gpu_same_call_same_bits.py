"""The result of a call is a function of its arguments: not of the batches the context has seen before, and not of
whether the call is replayed from a captured graph."""
import pytest
import torch

import workloads as wl

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2503_06433_amd as ss
    from paper_2503_06433_amd.harness import make_context, pp_desc, tp_desc, torch_dtype, empty_like_acts


def _filled(gen, shape, dtype, std=1.0):
    return torch.empty(shape, device="cuda", dtype=torch_dtype(dtype)).normal_(0, std, generator=gen)


def test_rows_beyond_the_workspace_do_not_depend_on_an_earlier_smaller_batch():
    """2450 rows on a narrow shard (1280 x 8192): with a workspace for partial sums the contraction could be cut, and
    the workspace is there only once a batch of up to 2048 rows has run."""
    cfg = wl.ModelCfg(hidden=8192, n_q_heads=64, n_kv_heads=8, head_dim=128, ffn=512, n_layers=1, dtype=wl.BF16)
    T = 2450
    gen = torch.Generator(device="cuda").manual_seed(941)
    H, q, kv = cfg.hidden, 64 * 128, 8 * 128
    w = {n: _filled(gen, s, cfg.dtype, 0.02) for n, s in (("wq", (H, q)), ("wk", (H, kv)), ("wv", (H, kv)), ("wo", (q, H)),
                                                          ("wg", (H, 512)), ("wu", (H, 512)), ("wd", (512, H)))}
    w["g1"] = w["g2"] = torch.ones(H, device="cuda", dtype=torch.bfloat16)
    x = _filled(gen, (T, H), cfg.dtype)
    d, res = tp_desc(cfg, 8, 0), []
    for before in (0, 100):
        ctx = make_context(cfg, pages=T + 8, max_seq_len=32)
        ctx.load_layer(d, 0, w, ss.SS_DEVICE)
        out = empty_like_acts(T, H, cfg.dtype)
        for n in ([before] if before else []) + [T]:
            ctx.layer_prefill(d, 0, ss.SS_ATTN, list(range(n)), [1] * n, [0] * n, x[:n], out[:n])
        torch.cuda.synchronize()
        res.append(out)
        ctx.destroy()
    assert torch.equal(res[0], res[1])


@pytest.mark.parametrize("dtype,hidden,phase", [(wl.BF16, 256, 1), (wl.BF16, 200, 2), (wl.F32, 256, 1), (wl.F32, 256, 2)])
def test_captured_call_on_rows_of_another_alignment(dtype, hidden, phase):
    """A graph is captured on rows that are not 16-byte aligned, after an eager call of the same batch on rows that
    are: the workspaces of both routes are there, and every replay gives the eager result."""
    cfg = wl.ModelCfg(hidden=hidden, n_q_heads=2, n_kv_heads=2, head_dim=64, ffn=256, n_layers=1, dtype=dtype)
    _, raws = wl.make_layer_weights(cfg, 951)
    ctx = make_context(cfg, pages=64, max_seq_len=64)
    d = pp_desc(cfg)
    ctx.load_layer(d, 0, raws)
    n, gen = 8, torch.Generator(device="cuda").manual_seed(952)
    ids, one, zero = list(range(n)), [1] * n, [0] * n
    flat = _filled(gen, (n * hidden + 8,), dtype)
    shift = 1 if dtype == wl.F32 else 2                     # four bytes
    x, y = flat[:n * hidden].view(n, hidden), flat[shift:shift + n * hidden].view(n, hidden)
    out, eager = empty_like_acts(n, hidden, dtype), empty_like_acts(n, hidden, dtype)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        ctx.layer_prefill(d, 0, phase, ids, one, zero, x, out, side.cuda_stream)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):
        ctx.layer_prefill(d, 0, phase, ids, one, zero, y, out, side.cuda_stream)
    torch.cuda.synchronize()
    for rep in range(3):
        flat.normal_(0, 1, generator=gen)
        g.replay()
        torch.cuda.synchronize()
        ctx.layer_prefill(d, 0, phase, ids, one, zero, y, eager)
        torch.cuda.synchronize()
        assert torch.equal(out, eager), "replay %d" % rep
    ctx.destroy()
