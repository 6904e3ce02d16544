"""The swap-in of a re-shard follows its swap-out sequence by sequence: caches of several copies each way arrive bit for bit,
whether the caches go by direct copies or, with a short sequence among them, through the pinned ring, with a second call queued
behind the first and with plain swaps in between."""
import numpy as np
import pytest
import torch

import workloads as wl

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2503_06433_amd as ss
    from paper_2503_06433_amd.harness import make_context, pp_desc, tp_desc, to_raw


@pytest.mark.parametrize("short", [None, 5])
def test_two_reshards_in_a_row_arrive_bit_for_bit(short):
    cfg = wl.ModelCfg(hidden=256, n_q_heads=4, n_kv_heads=4, head_dim=128, ffn=64, n_layers=3, dtype=wl.BF16)
    lens = [513, 1024, 777, 2000, 600, 1500, 900, 1100, 640, 1300]                   # 62 MB, three and more copies out
    if short:
        lens[3] = short
    L, nkv = cfg.n_layers, cfg.n_kv_heads
    ids, total = list(range(len(lens))), sum(lens)
    ctx = make_context(cfg, pages=2 * sum(-(-n // 16) for n in lens) + 4, tier_bytes=2 * total * 2 * nkv * 128 * 2 * L + (1 << 20),
                       pinned_bytes=64 << 20)
    pp, tp = pp_desc(cfg), tp_desc(cfg, 2, 1)
    gen = torch.Generator(device="cuda").manual_seed(991)
    for round_ in range(2):                                          # the second round with other contents in the same pages
        staging = torch.empty(total * 2 * nkv * 128 * L, device="cuda", dtype=torch.bfloat16).normal_(0, 1, generator=gen)
        raw, off, want = to_raw(staging, wl.BF16), 0, []
        for n in lens:
            want.append(raw[off:off + L * 2 * nkv * n * 128].reshape(L, 2, nkv, n, 128))
            off += want[-1].size
        ctx.kv_import_dev(pp, ids, lens, staging)
        ctx.kv_reshard(pp, tp, ids[:6])
        ctx.kv_swap(pp, ss.SS_OUT, ids[6:8])                          # a swap-out that nobody follows, then another followed one
        ctx.kv_reshard(pp, tp, ids[8:])
        ctx.kv_swap(tp, ss.SS_IN, ids[6:8])
        ctx.sync()
        for i in ids:
            for l in range(L):
                assert np.array_equal(ctx.kv_read(tp, i, l, 2), want[i][l][:, 2:4]), "sequence %d, layer %d" % (i, l)
        ctx.kv_free(pp, ids)
        ctx.kv_free(tp, ids)
        ctx.host_tier_release(ids)
    ctx.destroy()
