"""What is timed when this framework is made faster: one GPU's share of re-sharded inference, called as a serving
program calls it.

A case names a model shape, a storage type, a sharding and a batch; `prepare` builds the context, the weights and the
cached sequences that such a program holds, `run` takes one batch through the public calls, `work` counts the bytes
and operations that the batch cannot do without.  Everything random is drawn from the seed, except the sequence
lengths: those belong to the case (`lens_seed`), so that the work of a case is a fixed number."""
import math

import numpy as np
import torch

import paper_2503_06433_amd as ss

# hidden, query heads, kv heads, head dim, ffn, rotary base: the shapes of the framework's own configurations
SHAPES = {
    "tiny": (256, 4, 4, 64, 688),
    "7b": (4096, 32, 32, 128, 11008),
    "13b": (5120, 40, 40, 128, 13824),
    "70b": (8192, 64, 8, 128, 28672),
}
DTYPES = {"f32": (ss.SS_F32, torch.float32, 4), "bf16": (ss.SS_BF16, torch.bfloat16, 2), "f16": (ss.SS_F16, torch.float16, 2)}
PAGE = 16


def listed():
    return [
        # the whole tiny fp32 model, four prompts of 32 tokens and eight greedy steps with the tokens given: the
        # smallest calls there are, a chain of launches
        {"name": "generate_tiny_f32", "kind": "generate", "model": "tiny", "dtype": "f32", "k": 1, "layers": 2, "vocab": 512,
         "seqs": 4, "dist": "uniform", "lo": 32, "hi": 32, "lens_seed": 1001, "steps": 8},
        # eight users chatting with a two-layer stage of the 7B shape: embedding, layers, LM head, token after token
        {"name": "decode_7b_chat8", "kind": "decode", "model": "7b", "dtype": "bf16", "k": 1, "layers": 2, "vocab": 2048,
         "seqs": 8, "dist": "uniform", "lo": 64, "hi": 1500, "lens_seed": 11, "steps": 8},
        # consecutive decode steps of an offline batch, one 7B-shape layer
        {"name": "decode_7b_b256", "kind": "decode", "model": "7b", "dtype": "bf16", "k": 1, "layers": 1, "vocab": 0,
         "seqs": 256, "dist": "uniform", "lo": 512, "hi": 2560, "lens_seed": 2003, "steps": 6},
        # the same with one shard of four of the 13B shape: partial sums out, the phases are separate calls
        {"name": "decode_13b_tp4_b512", "kind": "decode", "model": "13b", "dtype": "bf16", "k": 4, "layers": 1, "vocab": 0,
         "seqs": 512, "dist": "uniform", "lo": 256, "hi": 4096, "lens_seed": 3003, "steps": 6},
        # one shard of eight of the 70B shape (grouped queries, one kv head), a thousand sequences
        {"name": "decode_70b_tp8_b1024", "kind": "decode", "model": "70b", "dtype": "bf16", "k": 8, "layers": 1, "vocab": 0,
         "seqs": 1024, "dist": "uniform", "lo": 512, "hi": 4096, "lens_seed": 4003, "steps": 6},
        # one prompt of odd length: the first token's latency
        {"name": "prefill_7b_one_prompt", "kind": "prefill", "model": "7b", "dtype": "bf16", "k": 1, "layers": 1, "vocab": 0,
         "seqs": 1, "dist": "uniform", "lo": 333, "hi": 333, "lens_seed": 12, "steps": 1},
        # an ordinary prefill batch: 16 ragged prompts, 20 thousand tokens
        {"name": "prefill_7b_b16", "kind": "prefill", "model": "7b", "dtype": "bf16", "k": 1, "layers": 1, "vocab": 0,
         "seqs": 16, "dist": "uniform", "lo": 512, "hi": 2048, "lens_seed": 2002, "steps": 1},
        # IEEE half, 32 prompts of the 13B shape
        {"name": "prefill_13b_f16_b32", "kind": "prefill", "model": "13b", "dtype": "f16", "k": 1, "layers": 1, "vocab": 0,
         "seqs": 32, "dist": "uniform", "lo": 256, "hi": 2048, "lens_seed": 3002, "steps": 1},
        # two layers of the 70B-shape pipeline slice, 64 prompts of the offline length mix: the largest prefill
        {"name": "prefill_70b_slice_b64", "kind": "prefill", "model": "70b", "dtype": "bf16", "k": 1, "layers": 2, "vocab": 0,
         "seqs": 64, "dist": "lognormal", "lo": 128, "hi": 4096, "lens_seed": 5002, "steps": 1},
        # chunked prefill: two consecutive chunks of a prompt, each in one batch with 96 decoding sequences
        {"name": "mixed_7b_chunk768", "kind": "mixed", "model": "7b", "dtype": "bf16", "k": 1, "layers": 1, "vocab": 0,
         "seqs": 97, "dist": "uniform", "lo": 512, "hi": 2560, "lens_seed": 13, "steps": 2, "chunk": 768},
        # the repack kernels in both directions: the caches of 64 prompts over the ten layers of the slice come from
        # heads-major staging into pages and go out again
        {"name": "pages_70b_slice_b64", "kind": "pages", "model": "70b", "dtype": "bf16", "k": 1, "layers": 10, "vocab": 0,
         "seqs": 64, "dist": "lognormal", "lo": 128, "hi": 4096, "lens_seed": 5002, "steps": 1},
        # the switch between the two strategies: shard 0 of 4 of the weights and the caches of 16 prompts cross the
        # host, then the shard decodes its first token
        {"name": "switch_7b_tp4", "kind": "switch", "model": "7b", "dtype": "bf16", "k": 4, "layers": 1, "vocab": 0,
         "seqs": 16, "dist": "uniform", "lo": 512, "hi": 2048, "lens_seed": 2002, "steps": 1},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges: kinds by how often a serving program makes them, sizes over their logarithm."""
    kind = rng.choices(["decode", "prefill", "mixed", "generate", "pages", "switch"], [36, 28, 14, 8, 8, 6])[0]
    c = {"kind": kind, "model": "7b", "dtype": rng.choices(["bf16", "f16"], [4, 1])[0], "k": 1, "layers": 1, "vocab": 0,
         "seqs": 1, "dist": "uniform", "lo": 1, "hi": 1, "lens_seed": rng.randrange(1 << 20), "steps": 1}
    if kind == "generate":
        c.update(model="tiny", dtype="f32", layers=2, vocab=rng.choice([512, 500, 2048]), seqs=_log_int(rng, 1, 16),
                 lo=_log_int(rng, 1, 64), steps=rng.randint(2, 12))
        c["hi"] = c["lo"] + rng.randint(0, 64)
    elif kind == "decode":
        c["model"], c["k"] = rng.choice([("7b", 1), ("7b", 1), ("7b", 4), ("13b", 1), ("13b", 4), ("70b", 8), ("70b", 8), ("70b", 4)])
        c["seqs"] = _log_int(rng, 1, 1024)
        c["hi"] = _log_int(rng, 96, 4000)
        c["lo"] = max(1, int(c["hi"] * rng.uniform(0.05, 0.9)))
        c["steps"] = rng.randint(5, 8)
        kv = 2 * SHAPES[c["model"]][2] // c["k"] * 128 * 2
        while c["seqs"] * (c["lo"] + c["hi"]) // 2 * kv > 7e9:          # the largest listed cache
            c["seqs"] = max(1, c["seqs"] // 2)
        if c["k"] == 1 and c["seqs"] <= 32 and rng.random() < 0.5:      # a chat step with its embedding and LM head
            c.update(layers=2, vocab=2048)
            c["hi"] = min(c["hi"], 2500)
            c["lo"] = min(c["lo"], c["hi"])
    elif kind == "prefill":
        c["model"] = rng.choice(["7b", "7b", "13b", "70b"])
        tokens = _log_int(rng, 24, 48000)
        c["hi"] = min(4096, _log_int(rng, 16, 4096), tokens)
        c["lo"] = max(1, int(c["hi"] * rng.uniform(0.1, 1.0)))
        c["seqs"] = max(1, min(256, 2 * tokens // (c["lo"] + c["hi"])))
    elif kind == "mixed":
        c["model"] = rng.choice(["7b", "7b", "13b"])
        c["chunk"] = _log_int(rng, 64, 2048)
        c["seqs"] = 1 + _log_int(rng, 2, 255)
        c["hi"] = _log_int(rng, 128, 2560)
        c["lo"] = max(1, int(c["hi"] * rng.uniform(0.1, 1.0)))
        c["steps"] = 2
    elif kind == "pages":
        c["model"], c["layers"] = rng.choice([("7b", 1), ("7b", 3), ("13b", 1), ("70b", 10)])
        c["seqs"] = _log_int(rng, 1, 64)
        c["hi"] = _log_int(rng, 32, 2048)
        c["lo"] = max(1, int(c["hi"] * rng.uniform(0.1, 1.0)))
    else:
        c["k"] = rng.choice([2, 4])
        c["seqs"] = _log_int(rng, 1, 16)
        c["hi"] = _log_int(rng, 128, 2048)
        c["lo"] = max(1, int(c["hi"] * rng.uniform(0.2, 1.0)))
    return c


def _lens(case):
    """Prompt lengths (prefill, generate) or cached tokens before the first step of every sequence."""
    g = np.random.default_rng(case["lens_seed"])
    if case["dist"] == "lognormal":      # the offline length mix
        v = np.clip(np.rint(g.lognormal(7.0, 0.6, size=case["seqs"])), case["lo"], case["hi"])
    else:
        v = g.integers(case["lo"], case["hi"] + 1, size=case["seqs"])
    return [int(x) for x in v]


class _Draw:
    """Normal values drawn on the GPU from one seed."""

    def __init__(self, seed, dtype):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(int(seed))
        self.dtype = dtype

    def __call__(self, *shape, std=1.0, mean=0.0):
        return torch.empty(shape, device="cuda", dtype=self.dtype).normal_(mean, std, generator=self.g)


def _weights(nrm, model):
    H, nq, nkv, d, F = SHAPES[model]
    w = {n: nrm(*s, std=0.02) for n, s in (("wq", (H, nq * d)), ("wk", (H, nkv * d)), ("wv", (H, nkv * d)), ("wo", (nq * d, H)),
                                          ("wg", (H, F)), ("wu", (H, F)), ("wd", (F, H)))}
    w["g1"], w["g2"] = nrm(H, std=0.02, mean=1.0), nrm(H, std=0.02, mean=1.0)
    return w


def _raw(t):
    t = t.cpu()
    return t.numpy() if t.dtype == torch.float32 else t.view(torch.int16).numpy().view(np.uint16)


def prepare(case, seed):
    H, nq, nkv, d, F = SHAPES[case["model"]]
    code, tdt, es = DTYPES[case["dtype"]]
    kind, k, L, lens = case["kind"], case["k"], case["layers"], _lens(case)
    nrm = _Draw(seed, tdt)
    new = {"mixed": case.get("chunk", 0) * case["steps"], "prefill": 0, "pages": 0}.get(kind, case["steps"]) + 1
    pages = 2 * len(lens) + sum(-(-n // PAGE) for n in lens) + case["seqs"] * (-(-case["steps"] // PAGE) + 1) + -(-new // PAGE)
    tier = sum(lens) * 2 * nkv * d * es * L + (1 << 20) if kind == "switch" else 0
    ctx = ss.Context(ss.ModelCfg(H, nq, nkv, d, F, L, case["vocab"], 1e-5, 10000.0, code, PAGE),
                     ss.RuntimeCfg(pages, tier, (4 * 34 << 20) if tier else 0, 0, max(lens) + new + 8))
    pp = ss.ShardDesc(ss.SS_PP, 1, 0, 0, L)
    tp = ss.ShardDesc(ss.SS_TP, k, 0, 0, L)
    s = {"case": case, "ctx": ctx, "pp": pp, "tp": tp, "ids": list(range(1, len(lens) + 1)), "lens": lens,
         "stream": torch.cuda.current_stream().cuda_stream}
    desc = s["desc"] = tp if kind == "decode" else pp
    if kind != "pages":
        for l in range(L):
            w = _weights(nrm, case["model"])
            if kind == "switch":
                ctx.host_weights_put(l, w, ss.SS_DEVICE)
            else:
                ctx.load_layer(desc, l, w, ss.SS_DEVICE)
    if case["vocab"]:
        ctx.load_head(_raw(nrm(case["vocab"], H)), _raw(nrm(H, std=0.02, mean=1.0)), _raw(nrm(H, case["vocab"], std=0.02)))
        n_tok = sum(lens) if kind == "generate" else 0
        ids = torch.randint(0, case["vocab"], (n_tok + len(lens) * case["steps"],), device="cuda", generator=nrm.g).cpu().numpy()
        s["prompt"], s["tokens"] = ids[:n_tok].astype(np.int32), ids[n_tok:].astype(np.int32).reshape(case["steps"], len(lens))

    def act(*shape):
        return torch.empty(shape, device="cuda", dtype=tdt)

    B, T, steps = len(lens), sum(lens), case["steps"]
    if kind in ("decode", "mixed", "pages", "switch"):       # sequences whose cache is there already
        staging = nrm(T * 2 * (nkv // (k if kind == "decode" else 1)) * d * L)
        if kind == "pages":
            s["staging"], s["out"] = staging, torch.empty_like(staging)
        else:
            ctx.kv_import_dev(desc, s["ids"], lens, staging)
            torch.cuda.synchronize()
    if kind == "generate":
        s["x"], s["y"], s["xd"], s["yd"] = act(T, H), act(T, H), act(B, H), [act(B, H) for _ in range(steps)]
        s["logits"] = [torch.empty((B, case["vocab"]), device="cuda") for _ in range(steps + 1)]
        s["last"] = torch.tensor(np.cumsum(lens) - 1, device="cuda")
    elif kind == "prefill":
        s["x"], s["y"] = nrm(T, H), act(T, H)
    elif kind == "mixed":
        s["x"] = nrm(steps, B - 1 + case["chunk"], H)
        s["y"] = torch.empty_like(s["x"])
    elif kind == "decode":
        s["x"], s["y"] = nrm(steps, B, H), act(steps, B, H)
        if k > 1:
            s["x1"], s["y1"] = nrm(steps, B, H), act(steps, B, H)
        if case["vocab"]:
            s["logits"] = [torch.empty((B, case["vocab"]), device="cuda") for _ in range(steps)]
    elif kind == "switch":
        s["x"], s["y"], s["x1"], s["y1"] = nrm(B, H), act(B, H), nrm(B, H), act(B, H)
    return s


def run(s):
    return globals()["_run_" + s["case"]["kind"]](s)


def _run_generate(s):
    """Prompts in, `steps` tokens per sequence out, the sequences leave."""
    ctx, d, ids, lens, st = s["ctx"], s["desc"], s["ids"], s["lens"], s["stream"]
    n = len(ids)
    ctx.embed(s["prompt"], s["x"], st)
    ctx.layers_prefill(d, ids, lens, [0] * n, s["x"], s["y"], st)
    ctx.lm_head(s["y"].index_select(0, s["last"]), n, s["logits"][0], st)
    for i in range(s["case"]["steps"]):
        ctx.embed(s["tokens"][i], s["xd"], st)
        ctx.layers_decode(d, ids, [v + i for v in lens], s["xd"], s["yd"][i], st)
        ctx.lm_head(s["yd"][i], n, s["logits"][i + 1], st)
    ctx.kv_free(d, ids)
    return s["logits"], s["yd"]


def _run_decode(s):
    """`steps` consecutive tokens of every sequence."""
    ctx, d, ids, lens, st = s["ctx"], s["desc"], s["ids"], s["lens"], s["stream"]
    x, y = s["x"], s["y"]
    for i in range(s["case"]["steps"]):
        at = [v + i for v in lens]
        if s["case"]["vocab"]:
            ctx.embed(s["tokens"][i], x[i], st)
        if s["case"]["k"] == 1:
            ctx.layers_decode(d, ids, at, x[i], y[i], st)
        else:            # the two partial sums of a shard: the caller reduces them over the shards in between
            ctx.layer_decode(d, 0, ss.SS_ATTN, ids, at, x[i], y[i], st)
            ctx.layer_decode(d, 0, ss.SS_MLP, ids, at, s["x1"][i], s["y1"][i], st)
        if s["case"]["vocab"]:
            ctx.lm_head(y[i], len(ids), s["logits"][i], st)
    return (y, s.get("y1"), s.get("logits"))


def _run_prefill(s):
    ctx, d, ids, st = s["ctx"], s["desc"], s["ids"], s["stream"]
    ctx.layers_prefill(d, ids, s["lens"], [0] * len(ids), s["x"], s["y"], st)
    ctx.kv_free(d, ids)
    return s["y"]


def _run_mixed(s):
    """Consecutive chunks of the first sequence's prompt, each together with one token of all the others."""
    ctx, d, ids, lens, st = s["ctx"], s["desc"], s["ids"], s["lens"], s["stream"]
    chunk = s["case"]["chunk"]
    q = [chunk] + [1] * (len(ids) - 1)
    for i in range(s["case"]["steps"]):
        ctx.layer_prefill(d, 0, ss.SS_BOTH, ids, q, [v + i * n for v, n in zip(lens, q)], s["x"][i], s["y"][i], st)
    return s["y"]


def _run_pages(s):
    ctx, d, ids, st = s["ctx"], s["desc"], s["ids"], s["stream"]
    ctx.kv_import_dev(d, ids, s["lens"], s["staging"], st)
    ctx.kv_export_dev(d, ids, s["out"], st)
    ctx.kv_free(d, ids)
    return s["out"]


def _run_switch(s):
    ctx, pp, tp, ids, lens, st = s["ctx"], s["pp"], s["tp"], s["ids"], s["lens"], s["stream"]
    ctx.reshard_weights(None, tp, st)
    ctx.kv_reshard(pp, tp, ids, st)
    ctx.sync()
    ctx.layer_decode(tp, 0, ss.SS_ATTN, ids, lens, s["x"], s["y"], st)
    ctx.layer_decode(tp, 0, ss.SS_MLP, ids, lens, s["x1"], s["y1"], st)
    ctx.kv_free(tp, ids)
    ctx.host_tier_release(ids)
    return s["y"], s["y1"]


def work(case):
    """Weights once per layer call, cached keys and values once per step that attends to them, activations in and
    out; operations of the products and of causal attention."""
    H, nq, nkv, d, F = SHAPES[case["model"]]
    es = DTYPES[case["dtype"]][2]
    kind, k, L, V, lens, steps = case["kind"], case["k"], case["layers"], case["vocab"], _lens(case), case["steps"]
    W = (H * (nq + 2 * nkv) * d + nq * d * H + 3 * H * F) // k
    tok_kv = 2 * nkv // k * d * es                           # one token's keys and values in one layer
    B, T = len(lens), sum(lens)
    if kind == "pages":
        return {"bytes": 4.0 * T * tok_kv * L, "flops": 0.0}
    calls = []                                               # (new tokens, cached tokens before) per sequence of a call
    if kind in ("prefill", "generate"):
        calls.append([(n, 0) for n in lens])
    if kind in ("decode", "generate", "switch"):
        calls += [[(1, n + i) for n in lens] for i in range(steps)]
    if kind == "mixed":
        q = [case["chunk"]] + [1] * (B - 1)
        calls += [[(a, n + i * a) for n, a in zip(lens, q)] for i in range(steps)]
    by, fl = 0.0, 0.0
    for c in calls:
        t = sum(a for a, _ in c)
        pairs = sum(a * b + a * (a + 1) / 2 for a, b in c)
        by += L * (W * es + sum(b for _, b in c) * tok_kv + t * tok_kv) + 2 * t * H * es * (2 if k > 1 else 1)
        fl += L * (2.0 * W * t + 4.0 * nq // k * d * pairs)
        if V:
            by += H * V * es + B * V * 4 + B * H * es
            fl += 2.0 * B * H * V
    if kind == "switch":                                     # out: whole caches; in: the shard's heads and weights
        by += 2.0 * T * tok_kv * k * L + 2.0 * T * tok_kv * L + 2.0 * W * es * L
    return {"bytes": by, "flops": fl}


def tolerance(case):
    if case["kind"] == "pages":
        return "exact"                                       # movement only
    return {"f32": {"rel": 1e-5}, "bf16": {"rel": 1.5e-2}, "f16": {"rel": 2.5e-3}}[case["dtype"]]
