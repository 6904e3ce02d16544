"""Device-side import and export queued one behind the other without a wait: more calls than there are metadata images,
each with more pages than the one before, every byte back where it came from."""
import pytest
import torch

import workloads as wl

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2503_06433_amd.harness import make_context, pp_desc, torch_dtype


@pytest.mark.parametrize("dtype,nkv,d,layers", [(wl.BF16, 2, 128, 3), (wl.F32, 1, 64, 2)])
def test_queued_imports_and_exports_return_every_byte(dtype, nkv, d, layers):
    cfg = wl.ModelCfg(hidden=128, n_q_heads=nkv, n_kv_heads=nkv, head_dim=d, ffn=64, n_layers=layers, dtype=dtype)
    sets = [[1], [17, 16, 15], [700, 33, 1, 128], [2000] + list(range(1, 200)), [5, 4000]]
    ctx = make_context(cfg, pages=sum(-(-n // 16) for lens in sets for n in lens) + 4, max_seq_len=4096)
    desc = pp_desc(cfg)
    gen = torch.Generator(device="cuda").manual_seed(921)
    src, dst, ids = [], [], []
    for j, lens in enumerate(sets):
        src.append(torch.randint(-30000, 30000, (sum(lens) * 2 * nkv * d * layers,), device="cuda", generator=gen).to(torch_dtype(dtype)))
        dst.append(torch.full_like(src[-1], 3.0))
        ids.append([1000 * j + i for i in range(len(lens))])
    for j, lens in enumerate(sets):
        ctx.kv_import_dev(desc, ids[j], lens, src[j])
    for _ in range(2):
        for j in range(len(sets)):
            ctx.kv_export_dev(desc, ids[j], dst[j])
    torch.cuda.synchronize()
    for j in range(len(sets)):
        assert torch.equal(src[j], dst[j]), "set %d" % j
    ctx.destroy()
