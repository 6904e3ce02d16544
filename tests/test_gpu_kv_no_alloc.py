"""Device-side import and export allocate nothing: the first call of a context, and calls with more and more metadata
(up to the 32768 units of one launch), leave the free device memory as it was."""
import pytest
import torch

import workloads as wl

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2503_06433_amd.harness import make_context, pp_desc, torch_dtype


def test_import_and_export_allocate_nothing():
    layers, sizes = 20, [1, 16, 250, 2000]
    cfg = wl.ModelCfg(hidden=64, n_q_heads=1, n_kv_heads=1, head_dim=64, ffn=64, n_layers=layers, dtype=wl.BF16)
    ctx = make_context(cfg, pages=2 * max(sizes) + 4, max_seq_len=64)
    desc = pp_desc(cfg)
    assert ctx.kv_free_pages(desc) == 2 * max(sizes) + 4
    per = 2 * 64 * layers
    src = torch.randint(-30000, 30000, (20 * max(sizes) * per,), device="cuda").to(torch_dtype(wl.BF16))
    dst = torch.full_like(src, 3.0)
    ctx.kv_import_dev(desc, [10 ** 6], [1], src)             # the page pools, and the kernels' code
    ctx.kv_export_dev(desc, [10 ** 6], dst)
    ctx.kv_free(desc, [10 ** 6])
    torch.cuda.synchronize()

    def unchanged(call, what):
        free = torch.cuda.mem_get_info()[0]
        call()
        assert torch.cuda.mem_get_info()[0] == free, what

    for n in sizes:
        ids = list(range(n))
        unchanged(lambda: ctx.kv_import_dev(desc, ids, [20] * n, src), "import of %d sequences" % n)
        dst.fill_(3.0)
        unchanged(lambda: ctx.kv_export_dev(desc, ids, dst), "export of %d sequences" % n)
        torch.cuda.synchronize()
        assert torch.equal(dst[:20 * n * per], src[:20 * n * per])
        ctx.kv_free(desc, ids)
    ctx.destroy()
