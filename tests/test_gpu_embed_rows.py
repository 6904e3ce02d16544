"""Embedding rows: token ids that travel as kernel arguments, around the size of a launch and of the path that copies them."""
import numpy as np
import pytest
import torch

import workloads as wl

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2503_06433_amd.harness import make_context, to_device


@pytest.mark.parametrize("dtype,hidden", [(wl.F32, 36), (wl.BF16, 200), (wl.BF16, 132)])
def test_embedding_rows_around_the_size_of_a_launch(dtype, hidden):
    vocab = 97
    cfg = wl.ModelCfg(hidden=hidden, n_q_heads=1, n_kv_heads=1, head_dim=64, ffn=64, n_layers=1, dtype=dtype, vocab=vocab)
    raws = wl.make_head_weights(cfg, 914)[1]
    table = raws["embed"]
    ctx = make_context(cfg, pages=4, max_seq_len=32)
    ctx.load_head(table, raws["gf"], raws["wlm"])
    rng = np.random.default_rng(917)
    for n in (1, 511, 512, 513, 2048, 2049):
        ids = rng.integers(0, vocab, size=n).astype(np.int32)
        want = to_device(table[ids], dtype)
        flat = torch.zeros((n + 1) * hidden + 1, device="cuda", dtype=want.dtype)
        for off in (0, 1):                                    # 16-byte aligned rows, and not
            flat.fill_(7.0)
            out = flat[off:off + (n + 1) * hidden].view(n + 1, hidden)
            sent = ids.copy()
            ctx.embed(sent, out)
            sent[:] = 0                                       # the ids are the caller's again once the call is back
            torch.cuda.synchronize()
            assert torch.equal(out[:n], want) and (out[n] == 7.0).all()
    ctx.destroy()
