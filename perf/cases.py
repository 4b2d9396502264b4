"""The performance cases of this repository: what a user of the library has it do, through its public entry points.

A case names an operation and its sizes.  The model shapes are keep_synth's (the 7B, 14B and 32B decoders and the
fp32 "tiny" one), the prompts are those of its workloads or lie between them.  Inputs are random draws of the
distributions the path meets: weights N(0, 0.02) with smaller residual projections, embeddings N(0, 1), RMSNorm
weights around 1, QKV biases, group caches with the standard deviation of projected keys and values.
"""
import math

import numpy as np
import torch

import keep_synth as ks
from paper_2602_23592_amd import KeepContext, KeepPrompt
from paper_2602_23592_amd import binding as kb

MODELS = {"tiny": ks.WORKLOADS["tiny"].shape, "7b": ks.WORKLOADS["qwen7b_16k"].shape,
          "14b": ks.WORKLOADS["qwen14b_32k"].shape, "32b": ks.WORKLOADS["qwen32b_32k_host"].shape}
BUDGETS = {"groups": kb.KEEP_BUDGET_GROUP_COUNT, "tokens": kb.KEEP_BUDGET_TOKENS}


def _prefill(name, model, layers, groups, instr, ratio, hops, budget="groups", kv="device", schedule="linear"):
    """groups: (count, shortest, longest) of the memories in prompt order, static groups first.  schedule: the ratio
    falls from layer to layer ("linear") or in three steps ("steps": fewer selections among many memories)."""
    (n1, a1, b1), (n2, a2, b2) = (groups + [(0, 1, 1)])[:2]
    return {"name": name, "op": "prefill", "model": model, "layers": layers, "n1": n1, "lo1": a1, "hi1": b1, "n2": n2,
            "lo2": a2, "hi2": b2, "instr": instr, "ratio": ratio, "hops": hops, "budget": budget, "kv": kv,
            "schedule": schedule}


def listed():
    return [
        # the smallest whole prefill: fp32 storage, 2 layers, 1 088 tokens (what a first test or a small model runs)
        _prefill("prefill_tiny_f32", "tiny", 2, [(8, 128, 128)], 64, 0.15, 1),
        # a short bf16 prompt, a few retrieved memories and one sentence: latency, launches, weights read once
        _prefill("prefill_7b_short", "7b", 28, [(9, 20, 61)], 33, 0.3, 2),
        # an ordinary planning prompt (64 memories, 16 640 tokens)
        _prefill("prefill_7b_16k", "7b", 28, [(64, 256, 256)], 256, 0.15, 2),
        # the headline prompt: 16 static groups, 256 dynamic segments, 33 024 tokens, budget in tokens
        _prefill("prefill_14b_33k", "14b", 48, [(16, 1024, 1024), (256, 64, 64)], 256, 0.10, 3, "tokens"),
        # the largest prompt: 1 024 ragged memories, about 65 800 tokens
        _prefill("prefill_14b_66k", "14b", 48, [(1024, 32, 96)], 256, 0.10, 3, schedule="steps"),
        # group caches in pinned host memory, loaded layer by layer beside the compute (a quarter of the 32B depth)
        _prefill("prefill_32b_host", "32b", 16, [(128, 128, 384)], 256, 0.10, 2, kv="pinned"),
        # pure reuse of a long cache by a 16-token instruction: re-alignment, weight streaming, row-sparse attention
        _prefill("reuse_14b_16rows", "14b", 48, [(16, 1024, 1024), (256, 64, 64)], 16, 0.0, 1),
        # the answer: first token and 8 greedy tokens over the joined 33 024-token cache
        {"name": "decode_14b_33k", "op": "decode", "model": "14b", "layers": 48, "ctx": 33024, "new": 9, "int4": False},
        # the same with INT4 weight-only projections on the shape they are meant for (a quarter of its depth)
        {"name": "decode_32b_int4", "op": "decode", "model": "32b", "layers": 16, "ctx": 33024, "new": 17, "int4": True},
        # memory update: one dynamic segment of 64 tokens is cached on its own
        {"name": "unit_14b_64", "op": "units", "model": "14b", "layers": 48, "count": 1, "lo": 64, "hi": 64, "int4": False},
        # memory update: a static group turned dynamic, its ragged segments cached each on its own in one pass
        {"name": "units_14b_ragged", "op": "units", "model": "14b", "layers": 48, "count": 16, "lo": 24, "hi": 105,
         "int4": False},
        # the selection alone, on device-resident scores, as many candidates as the largest prompt has memories
        {"name": "select_1024", "op": "select", "m": 1024, "ratio": 0.15, "hops": 3, "budget": "groups"},
    ]


def draw(rng):
    """One more case of the ranges above; sizes log-uniform, odd ones included."""
    def logint(lo, hi):
        return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))

    limit = max(_cost(c) for c in listed())
    while True:
        op = rng.choice(["prefill", "prefill", "prefill", "reuse", "decode", "units", "units", "select"])
        model = rng.choice(["7b", "14b", "32b"])
        layers = logint(4, {"7b": 28, "14b": 48, "32b": 16}[model])
        if op == "prefill" or op == "reuse":
            if op == "prefill" and rng.random() < 0.2:
                model, layers = "tiny", 2
            mean = logint(24, 512)
            tokens = logint(300, 4096 if model == "tiny" else 40000)
            n = max(2, min(1024, tokens // mean))
            lo = max(1, mean - rng.randrange(mean // 2 + 1))
            c = _prefill("", model, layers, [(n, lo, 2 * mean - lo)], logint(1, 300) if op == "prefill" else logint(1, 64),
                         round(rng.uniform(0.05, 0.3), 3) if op == "prefill" else 0.0, rng.randint(1, 4),
                         rng.choice(["groups", "tokens"]), "pinned" if rng.random() < 0.2 else "device",
                         "linear" if n <= 128 else "steps")
        elif op == "decode":
            c = {"op": "decode", "model": model, "layers": layers, "ctx": logint(300, 40000), "new": rng.randint(2, 20),
                 "int4": rng.random() < 0.5}
        elif op == "units":
            lo = logint(1, 300)
            c = {"op": "units", "model": model, "layers": layers, "count": rng.choice([1, 1, 1, rng.randint(2, 20)]),
                 "lo": lo, "hi": lo + rng.randrange(lo + 1), "int4": rng.random() < 0.3}
        else:
            c = {"op": "select", "m": logint(9, 4000), "ratio": round(rng.uniform(0.03, 0.4), 3), "hops": rng.randint(1, 4),
                 "budget": rng.choice(["groups", "tokens"])}
        c.pop("name", None)
        if _cost(c) <= limit:
            return c


# ---------------------------------------------------------------------------------------------------------------
# layouts (a function of the case alone, so that every seed has the same shapes)
# ---------------------------------------------------------------------------------------------------------------
def _shape(case):
    m = MODELS[case["model"]]
    return ks.ModelShape(case["layers"], m.hidden, m.n_q_heads, m.n_kv_heads, m.head_dim, m.ffn_dim, m.vocab,
                         m.rope_theta, m.rms_eps, m.storage)


def _lens(case):
    r = np.random.Generator(np.random.PCG64(1))
    parts = [r.integers(case["lo" + i], case["hi" + i] + 1, size=case["n" + i]) for i in "12"]
    return [int(v) for p in parts for v in p]


def _unit_lens(case):
    r = np.random.Generator(np.random.PCG64(2))
    return [int(v) for v in r.integers(case["lo"], case["hi"] + 1, size=case["count"])]


def _schedule(case):
    L = case["layers"]
    r = ks.ratio_schedule(case["ratio"], L)
    if case["schedule"] == "steps":
        for l in range(1, L):
            r[l] = case["ratio"] * (1.5, 1.0, 0.5)[(l - 1) * 3 // (L - 1)]
    if case["ratio"] == 0.0:
        r[0] = 0.0          # pure reuse: no memory is recomputed at any layer
    return r


# ---------------------------------------------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------------------------------------------
def _normal(gen, dtype, std, *size):
    return torch.empty(size, dtype=dtype, device="cuda").normal_(0.0, std, generator=gen)


def _residual_scale(s, name):
    """Projections that add to the residual stream start smaller the deeper the decoder is, as is usual."""
    return 1.0 / math.sqrt(2 * s.n_layers) if name in ("wo", "wdown") else 1.0


def _token_ids(host, lens, vocab):
    """Every memory (and the instruction) speaks of a few things of its own: its tokens are draws from three."""
    return np.concatenate([host.choice(host.integers(0, vocab, size=3), size=n) for n in lens]).astype(np.int32)


def _weights(s, gen, dtype, int4):
    layers, layers4 = [], []
    shapes = ks.layer_weight_shapes(s)
    for _ in range(s.n_layers):
        w = {}
        if int4:
            w4 = {}
            for n in ks.INT4_MATS:
                rows, k = shapes[n]
                codes = torch.randint(0, 256, (rows * k // 2,), generator=gen, device="cuda", dtype=torch.uint8)
                zero = torch.randint(7, 9, (rows * k // ks.INT4_GROUP,), generator=gen, device="cuda", dtype=torch.int32)
                scale = torch.rand((rows * k // ks.INT4_GROUP,), generator=gen, device="cuda").mul_(0.5).add_(0.75)
                scale *= 0.02 * _residual_scale(s, n) / 4.6         # (uniform codes have a standard deviation of 4.6)
                bits = scale.to(torch.bfloat16).view(torch.int16).to(torch.int32) & 0xFFFF
                w4[n] = (codes, (bits | (zero << 16)).contiguous())
                w[n] = kb.dequantize_int4(*w4[n], rows, k)
            layers4.append(w4)
        else:
            for n in ks.INT4_MATS:
                w[n] = _normal(gen, dtype, 0.02 * _residual_scale(s, n), *shapes[n])
        for n in ("ln1", "ln2"):
            w[n] = _normal(gen, dtype, 0.1, s.hidden).add_(1.0)
        for n, d in (("bq", s.q_dim), ("bk", s.kv_dim), ("bv", s.kv_dim)):
            w[n] = _normal(gen, dtype, 0.02, d)
        layers.append(w)
    return layers, layers4


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    host = np.random.Generator(np.random.PCG64(int(seed)))
    if case["op"] == "select":
        return _prepare_select(case, gen, host)
    s = _shape(case)
    dtype = ks.torch_dtype(s.storage)
    st = {"case": case, "shape": s}
    layers, layers4 = _weights(s, gen, dtype, case.get("int4", False))
    embed = _normal(gen, dtype, 1.0, s.vocab, s.hidden)
    kv_std = 0.02 * math.sqrt(s.hidden)       # standard deviation of a projected key or value
    if case["op"] == "prefill":
        lens = _lens(case)
        groups, n = len(lens), sum(lens) + case["instr"]
        ids = _token_ids(host, lens + [case["instr"]], s.vocab)
    elif case["op"] == "decode":
        groups, n = 1, case["ctx"] + case["new"]
    else:
        lens = _unit_lens(case)
        groups, n = 1, sum(lens)
        ids = _token_ids(host, lens, s.vocab)
    st["ctx"] = KeepContext(s, layers, embed, n, groups, kb.KEEP_KERNELS_AUTO, *[torch.cuda.Stream() for _ in range(3)])
    if layers4:
        st["ctx"].attach_int4(layers4)
    row = (s.n_kv_heads, s.head_dim)
    if case["op"] == "prefill":
        n_mem = sum(lens)
        k_all, v_all = (_normal(gen, dtype, kv_std, s.n_layers, n_mem, *row) for _ in range(2))
        where = kb.KEEP_KV_DEVICE
        if case["kv"] == "pinned":
            where = kb.KEEP_KV_PINNED_HOST
            k_dev, v_dev = k_all, v_all
            k_all, v_all = (torch.empty(k_dev.shape, dtype=dtype, pin_memory=True) for _ in range(2))
            k_all.copy_(k_dev)
            v_all.copy_(v_dev)
            del k_dev, v_dev
        off = np.concatenate([[0], np.cumsum(lens)])
        blocks = [[[t[l, off[g]:off[g + 1]] for g in range(groups)] for l in range(s.n_layers)] for t in (k_all, v_all)]
        st["prompt"] = KeepPrompt(lens, case["instr"], ids, blocks[0], blocks[1], s.n_layers, where)
        st["ratios"] = _schedule(case)
        st["k"], st["v"] = (torch.zeros((s.n_layers, n, *row), dtype=dtype, device="cuda") for _ in range(2))
        st["x"] = torch.zeros((case["instr"], s.hidden), dtype=dtype, device="cuda")
    elif case["op"] == "decode":
        st["k"], st["v"] = (_normal(gen, dtype, kv_std, s.n_layers, n, *row) for _ in range(2))
        st["x"] = _normal(gen, dtype, 8.0, s.hidden)
        st["norm"] = _normal(gen, dtype, 0.1, s.hidden).add_(1.0)
        head = _normal(gen, dtype, 0.02, s.vocab, s.hidden)
        # a decisive head, as a trained model's: the row of each answer token points along what precedes it, so that
        # rounding never decides the greedy choice
        answer = host.choice(s.vocab, size=case["new"], replace=False)
        before = [st["x"]] + [embed[int(t)] for t in answer[:-1]]
        for t, e in zip(answer, before):
            e = e.float()
            head[int(t)] += (0.02 * math.sqrt(s.hidden) * e / e.norm()).to(dtype)
        st["head"] = head
        st["logits"] = torch.zeros((case["new"], s.vocab), dtype=torch.float32, device="cuda")
    else:
        st["lens"], st["ids"] = lens, ids
        st["k"], st["v"] = (torch.zeros((s.n_layers, n, *row), dtype=dtype, device="cuda") for _ in range(2))
    return st


def _prepare_select(case, gen, host):
    m = case["m"]
    # m candidates left of twice as many memories; attention of later memories to earlier ones (none forwards), the
    # instruction's row last, some memories more to the point than others
    S = torch.rand((m + 1, m), generator=gen, device="cuda", dtype=torch.float32).tril_(-1)
    S *= torch.randn((m,), generator=gen, device="cuda", dtype=torch.float32).exp_()
    groups = np.sort(host.choice(2 * m, size=m, replace=False)).astype(np.int32)
    lens = host.integers(32, 97, size=2 * m).astype(np.int32)
    return {"case": case, "S": S, "groups": torch.from_numpy(groups).cuda(), "len": torch.from_numpy(lens).cuda(),
            "mem_tokens": int(lens.sum()), "result": torch.zeros(m + 2, dtype=torch.int32, device="cuda")}


# ---------------------------------------------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------------------------------------------
def run(st):
    case = st["case"]
    if case["op"] == "select":
        kb.select_groups_static(st["S"], st["groups"], st["len"], st["mem_tokens"], case["ratio"], case["hops"],
                                BUDGETS[case["budget"]], kb.KEEP_SOURCES_QUERY_AND_SET, st["result"])
        return st["result"]
    ctx = st["ctx"]
    if case["op"] == "prefill":
        sets, _ = ctx.prefill(st["prompt"], st["ratios"], case["hops"], st["k"], st["v"], st["x"], BUDGETS[case["budget"]])
        member = np.zeros((len(sets), st["prompt"].n_groups), dtype=np.int32)   # the sets, as one array of a fixed shape
        for l, groups in enumerate(sets):
            member[l, groups] = 1
        return {"k": st["k"], "v": st["v"], "x": st["x"], "sets": member}
    if case["op"] == "decode":
        tokens = ctx.decode(st["norm"], st["head"], st["x"], st["k"], st["v"], case["ctx"], case["new"],
                            logits_out=st["logits"])
        written = slice(case["ctx"], case["ctx"] + case["new"] - 1)             # the rows of the tokens that were fed
        return {"tokens": np.asarray(tokens, dtype=np.int32), "logits": st["logits"], "k": st["k"][:, written],
                "v": st["v"][:, written]}
    if len(st["lens"]) == 1:
        ctx.precompute_group(st["ids"], st["k"], st["v"])
    else:
        ctx.precompute_groups(st["lens"], st["ids"], st["k"], st["v"])
    return {"k": st["k"], "v": st["v"]}


# ---------------------------------------------------------------------------------------------------------------
# what a pass cannot do without, and how far two correct implementations lie apart
# ---------------------------------------------------------------------------------------------------------------
def work(case):
    if case["op"] == "select":
        m = case["m"]
        return {"bytes": 4.0 * m * (m + 1) / 2 + 4.0 * m + 12.0 * m, "flops": 2.0 * m * m}
    s = _shape(case)
    e = 4 if s.storage == "f32" else 2
    qkv, out, ffn = s.hidden * (s.q_dim + 2 * s.kv_dim), s.q_dim * s.hidden, 3 * s.hidden * s.ffn_dim
    w_bytes = (qkv + out + ffn) * (0.5 + 4.0 / 128 if case.get("int4") else e)
    kv_row = 2 * s.kv_dim * e                                   # K and V of one row of one layer
    L = s.n_layers
    if case["op"] == "decode":
        fed = case["new"] - 1
        step = L * w_bytes + s.vocab * s.hidden * e + L * case["ctx"] * kv_row
        flops = 2.0 * L * (qkv + out + ffn) + 2.0 * s.vocab * s.hidden + 4.0 * L * s.q_dim * case["ctx"]
        return {"bytes": fed * step + s.vocab * s.hidden * e + 4.0 * case["new"] * s.vocab,
                "flops": fed * flops + 2.0 * s.vocab * s.hidden}
    if case["op"] == "units":
        lens = _unit_lens(case)
        n, pairs = sum(lens), sum(v * (v + 1) / 2 for v in lens)
        return {"bytes": (L - 1) * w_bytes + 2 * s.kv_dim * s.hidden * e + L * n * kv_row + n * s.hidden * e,
                "flops": 2.0 * n * ((L - 1) * (qkv + out + ffn) + 2 * s.kv_dim * s.hidden) + (L - 1) * 4.0 * s.q_dim * pairs}
    lens = _lens(case)
    n_mem, lq = sum(lens), case["instr"]
    n = n_mem + lq
    r = _schedule(case)
    rows = [float(r[l]) * n_mem + lq for l in range(L)]         # rows recomputed at each layer
    flops, nbytes = 0.0, L * w_bytes
    for l in range(L):
        kept = rows[l + 1] if l + 1 < L else lq                 # rows whose hidden state is read behind the layer
        flops += 2.0 * rows[l] * qkv + 2.0 * kept * (out + ffn)
        flops += 4.0 * s.q_dim * ((kept - lq) ** 2 / 2 + lq * n)  # their attention, at least: memories at the prompt's front
        if 0 < rows[l] - lq and l + 1 < L and case["ratio"] > 0:
            flops += 2.0 * s.q_dim * lq * (rows[l] - lq)        # scores of the instruction towards the candidates
        nbytes += (n - rows[l]) * kv_row + n * kv_row           # cached rows in, joined cache out
    return {"bytes": nbytes + rows[0] * s.hidden * e + lq * s.hidden * e, "flops": flops}


def _cost(case):
    w = work(case)
    return max(w["bytes"] / 4.0e12, w["flops"] / 1.0e15)


def tolerance(case):
    """Measured against the same passes with the hidden dimension permuted (every sum over it in another order) and
    against the generic kernels: fp32 rel 3e-7, max 2.5e-6; bf16 at full depth rel 2.4e-2, max 0.17 (rounding of the
    residual stream, layer after layer), and rel 1.5e-2 at 16 layers."""
    if case["op"] == "select":
        return "exact"
    if case["model"] == "tiny":
        return {"rel": 1.2e-6, "max": 1e-5}
    return {"rel": 3e-2, "max": 0.6}
