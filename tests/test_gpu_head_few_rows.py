"""Final norm and LM head of few rows in one product (bf16, fp32; IEEE half keeps them apart), against the CPU oracle and, for the
same rows, against the two-launch route that unaligned activations still take: row counts around the tiles of 16 rows, a
contraction of whole chunks, one that ends inside a chunk, more and fewer chunks than a block has waves."""
import numpy as np
import pytest
import torch

import workloads as wl
from oracle import layer_math as lm

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2503_06433_amd.harness import make_context, to_device, rel_err, tol, row_errs, ROW_TOL


@pytest.mark.parametrize("dtype,hidden,vocab", [
    (wl.BF16, 4096, 2048), (wl.BF16, 256, 500), (wl.BF16, 2120, 1001), (wl.F16, 512, 1024), (wl.F32, 256, 512), (wl.F32, 1044, 333),
])
def test_head_of_few_rows_matches_oracle(dtype, hidden, vocab):
    cfg = wl.ModelCfg(hidden=hidden, n_q_heads=1, n_kv_heads=1, head_dim=64, ffn=64, n_layers=1, vocab=vocab, dtype=dtype)
    hv, hr = wl.make_head_weights(cfg, 87)
    ctx = make_context(cfg, pages=4)
    ctx.load_head(hr["embed"], hr["gf"], hr["wlm"])
    for n in (1, 8, 9, 16, 17, 33, 48, 64, 65):
        xv, xr = wl.make_activations((n, hidden), 88 + n, dtype)
        ref = lm.lm_logits(cfg, hv, xv)
        x = to_device(xr, dtype)
        apart = torch.empty(x.numel() + 1, device="cuda", dtype=x.dtype)
        apart[1:] = x.reshape(-1)
        got = []
        for rows in (x, apart[1:]):
            logits = torch.full((n + 1, vocab), 7.0, device="cuda", dtype=torch.float32)
            ctx.lm_head(rows, n, logits)
            torch.cuda.synchronize()
            g = logits.cpu().numpy()
            assert (g[n] == 7.0).all()
            assert rel_err(g[:n], ref) <= tol(dtype)
            got.append(row_errs(g[:n], ref))
        assert max(got[0]) <= ROW_TOL[dtype], "%d rows" % n
        # one rounding of each scaled activation to the storage type either way
        assert np.median(got[0]) <= 1.2 * np.median(got[1]) + 1e-7, "%d rows: %.2e against %.2e" % (n, np.median(got[0]), np.median(got[1]))
    ctx.destroy()
