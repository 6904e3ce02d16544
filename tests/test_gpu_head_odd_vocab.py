"""LM head of vocabularies that are no multiple of eight (logit rows that are not whole 16-byte pieces), and of one with more
128-wide tiles than compute units, against the CPU oracle: the few-row kernel, and the register-staged one it hands over to, without a workspace for partial sums, with the layer
calls' workspace and with the fixed scratch of the call that allocates nothing (K whole and in two to eight ranges)."""
import pytest
import torch

import workloads as wl
from oracle import layer_math as lm

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2503_06433_amd as ss
    from paper_2503_06433_amd.harness import make_context, pp_desc, to_device, empty_like_acts, rel_err, tol


@pytest.mark.parametrize("dtype,hidden,vocab,rows", [
    (wl.BF16, 512, 1001, (5, 64, 65, 130, 300)),
    (wl.F16, 1024, 1001, (70,)),
    (wl.F16, 256, 24601, (8, 32, 33, 64, 65)),        # three and a few more rounds of few-row blocks
    (wl.BF16, 128, 49201, (8, 9, 16, 17)),            # five
    (wl.BF16, 128, 40000, (17, 64, 128, 129)),        # 313 tiles
])
def test_head_of_an_odd_vocabulary_matches_oracle(dtype, hidden, vocab, rows):
    cfg = wl.ModelCfg(hidden=hidden, n_q_heads=1, n_kv_heads=1, head_dim=64, ffn=64, n_layers=1, vocab=vocab, dtype=dtype)
    hv, hr = wl.make_head_weights(cfg, 971)
    _, raws = wl.make_layer_weights(cfg, 972)
    ctx = make_context(cfg, pages=8, max_seq_len=32)
    ctx.load_head(hr["embed"], hr["gf"], hr["wlm"])
    d = pp_desc(cfg)
    ctx.load_layer(d, 0, raws)
    ref = {n: lm.lm_logits(cfg, hv, wl.make_activations((n, hidden), 973 + n, dtype)[0]) for n in rows}
    for workspace in (False, True):
        if workspace:                                 # a layer call of few rows makes it
            one = empty_like_acts(1, hidden, dtype).zero_()
            ctx.layer_prefill(d, 0, ss.SS_MLP, [0], [1], [0], one, torch.empty_like(one))
        for n in rows:
            x = to_device(wl.make_activations((n, hidden), 973 + n, dtype)[1], dtype)
            for call in (ctx.lm_head, ctx.lm_head_noalloc):
                out = torch.full((n + 1, vocab), 7.0, device="cuda")
                call(x, n, out)
                torch.cuda.synchronize()
                got = out.cpu().numpy()
                assert (got[n] == 7.0).all()
                assert rel_err(got[:n], ref[n]) <= tol(dtype), "%d rows" % n
    ctx.destroy()
