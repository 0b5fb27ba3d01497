"""The work whose speed this framework answers for, as cases that can be timed and checked.

Every case goes through the public entry points of `paper_2604_02047_amd`, as a decoding program
calls them:

  layer   goose_embed + goose_verify_layer: the tree's rows enter one decoder layer.  One layer is
          nine tenths of what a pass over a deep model repeats; trees of 1 to 128 nodes, prefixes of
          16 to 16384 slots, multi-head and grouped-query models, bf16 and fp16 storage, both
          operand modes.
  head    goose_lm_head_argmax with logits and margins, then goose_harvest_topk: "verify and harvest",
          once per cycle.
  step    goose_verify_step replayed as a HIP graph: a whole cycle of a small model, logits included.
  batch   goose_verify_step_batched replayed as a HIP graph: several requests of a grouped-query model
          in one pass, every request with its own caches and successor tables.

Model dimensions are those of the repository's own shapes (Vicuna-7B/13B/33B, Llama-3-8B, Qwen3-8B and the
two-layer oracle-scale model).  Values are random: activations and keys of unit size, projections of
0.02, so that scores, softmax weights and SwiGLU inputs spread as they do in a trained model.  Whole
steps use an output head that favours the successor of a node's token (token + 1): predictions are
then decided by clear margins, planted drafts are accepted for a few nodes, and the walk and the commit
have work to do.
"""
import math

import numpy as np
import torch

import paper_2604_02047_amd as goose
from paper_2604_02047_amd.binding import GooseContext

#           layers of the real model are irrelevant here: hidden, heads, KV heads, head_dim, ffn, vocab, base, eps, q/k norm
MODELS = {
    "tiny": (256, 4, 4, 64, 688, 1024, 10000.0, 1e-5, False),
    "7b": (4096, 32, 32, 128, 11008, 32000, 10000.0, 1e-5, False),
    "13b": (5120, 40, 40, 128, 13824, 32000, 10000.0, 1e-5, False),
    "33b": (6656, 52, 52, 128, 17920, 32000, 10000.0, 1e-5, False),
    "llama3_8b": (4096, 32, 8, 128, 14336, 128256, 500000.0, 1e-5, False),
    "qwen3_8b": (4096, 32, 8, 128, 12288, 151936, 1000000.0, 1e-6, True),
}
BATCH_LAYERS = 8    # decoder layers of a batched pass: the head then weighs about as much as in a real stack
STEP_LAYERS = 2     # the two-layer oracle-scale model
HARVEST_K = 10      # successors kept per token (the paper's table width)
ACCEPTED = 3        # planted drafts that whole steps accept
DTYPES = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}
DEV = "cuda:0"


def listed():
    return [
        # a whole cycle of the fp32 model (CPU-oracle scale): nothing but launches and latency
        {"name": "step_tiny_f32_B8_P64", "kind": "step", "model": "tiny", "dtype": "f32", "two_term": False, "B": 8, "P": 64},
        # an autoregressive cycle (no draft found): one node
        {"name": "layer_7b_B1_P1024", "kind": "layer", "model": "7b", "dtype": "bf16", "two_term": False, "B": 1, "P": 1024},
        # the bypass: a matched chain of 20 tokens behind the anchor, fp16 storage as the paper runs it, short prompt
        {"name": "layer_7b_f16_B21_P333", "kind": "layer", "model": "7b", "dtype": "f16", "two_term": False, "B": 21, "P": 333},
        # the headline configuration: 64-node spine tree, prefix 1024
        {"name": "layer_7b_B64_P1024", "kind": "layer", "model": "7b", "dtype": "bf16", "two_term": False, "B": 64, "P": 1024},
        # grouped queries with q/k norm, a ragged tree in a ragged prefix
        {"name": "layer_qwen3_8b_B33_P1337", "kind": "layer", "model": "qwen3_8b", "dtype": "bf16", "two_term": False, "B": 33,
         "P": 1337},
        # the wide-range operand mode of the projections (two bf16 terms)
        {"name": "layer_llama3_8b_two_term_B61_P3001", "kind": "layer", "model": "llama3_8b", "dtype": "bf16", "two_term": True,
         "B": 61, "P": 3001},
        # the larger models of the paper at their tree budget
        {"name": "layer_13b_B80_P2048", "kind": "layer", "model": "13b", "dtype": "bf16", "two_term": False, "B": 80, "P": 2048},
        {"name": "layer_33b_B80_P4096", "kind": "layer", "model": "33b", "dtype": "bf16", "two_term": False, "B": 80, "P": 4096},
        # the stress configuration: the largest tree over a long context (also what a prefill chunk late in a prompt is)
        {"name": "layer_7b_B128_P16384", "kind": "layer", "model": "7b", "dtype": "bf16", "two_term": False, "B": 128, "P": 16384},
        # the output side of a cycle at a large vocabulary
        {"name": "head_llama3_8b_B64", "kind": "head", "model": "llama3_8b", "dtype": "bf16", "two_term": False, "B": 64, "P": 0},
        # the batch sweep of the paper: budget 32 per request; ragged sizes in the smaller one, the full 512 rows in the larger
        {"name": "batch_llama3_8b_8x30_P700", "kind": "batch", "model": "llama3_8b", "dtype": "bf16", "two_term": False, "n": 8,
         "B": 30, "P": 700},
        {"name": "batch_llama3_8b_16x32_P1024", "kind": "batch", "model": "llama3_8b", "dtype": "bf16", "two_term": False, "n": 16,
         "B": 32, "P": 1024},
    ]


def draw(rng):
    def log_int(lo, hi):
        return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))

    kind = rng.choice(["layer", "layer", "layer", "layer", "head", "batch", "batch", "step"])
    if kind == "step":
        return {"kind": kind, "model": "tiny", "dtype": "f32", "two_term": False, "B": log_int(1, 64), "P": log_int(1, 512)}
    model = rng.choice(["7b", "13b", "33b", "llama3_8b", "qwen3_8b"])
    dtype = rng.choice(["bf16", "bf16", "f16"])
    if kind == "layer":
        return {"kind": kind, "model": model, "dtype": dtype, "two_term": rng.random() < 0.2, "B": log_int(1, 128),
                "P": log_int(16, 16384)}
    if kind == "head":
        return {"kind": kind, "model": model, "dtype": dtype, "two_term": rng.random() < 0.2, "B": log_int(1, 128), "P": 0}
    # up to 512 stacked rows (every request padded to 32); the larger vocabulary and two-term operands with fewer of them
    model = rng.choice(["llama3_8b", "qwen3_8b"])
    two_term = rng.random() < 0.15
    B = rng.choice([rng.randint(4, 32), rng.randint(33, 64), 32])
    rows = 224 if two_term else (448 if model == "qwen3_8b" else 512)
    n = rng.randint(2, min(16, rows // (32 if B <= 32 else 64)))
    return {"kind": kind, "model": model, "dtype": "bf16", "two_term": two_term, "n": n, "B": B, "P": log_int(64, 1024)}


# ---- inputs: everything from the seed alone -------------------------------------------------------------
def _gen(seed, tag):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 1009 + tag)
    return g


def _randn(g, shape, std, dt):
    t = torch.empty(shape, dtype=dt, device=DEV)
    t.normal_(0.0, std, generator=g)
    return t


def _layer_weights(case, seed, l):
    """One layer's matrices as a checkpoint stores them, [out][in]."""
    H, nh, nkv, d, F = MODELS[case["model"]][:5]
    dt, g = DTYPES[case["dtype"]], _gen(seed, 100 + l)
    s = 0.02 * math.sqrt(4096.0 / H)
    w = {"wq": _randn(g, (nh * d, H), s, dt), "wk": _randn(g, (nkv * d, H), s, dt), "wv": _randn(g, (nkv * d, H), s, dt),
         "wo": _randn(g, (H, nh * d), s, dt), "wg": _randn(g, (F, H), s, dt), "wu": _randn(g, (F, H), s, dt),
         "wd": _randn(g, (H, F), 0.25 * s, dt)}
    for n, size in (("g1", H), ("g2", H), ("gq", d), ("gk", d)):
        w[n] = (1.0 + _randn(g, (size,), 0.1, torch.float32)).to(dt)
    return w


def _embedding(case, seed):
    return _randn(_gen(seed, 1), (MODELS[case["model"]][5], MODELS[case["model"]][0]), 1.0, DTYPES[case["dtype"]])


def _final_gain(case, seed):
    return (1.0 + _randn(_gen(seed, 2), (MODELS[case["model"]][0],), 0.1, torch.float32)).to(DTYPES[case["dtype"]])


def _successor_head(case, seed, embed):
    """An output head that favours token + 1: row v leans towards the embedding of v - 1, by as much as gives that word a
    probability of some tenths."""
    s = 0.02 * math.sqrt(4096.0 / MODELS[case["model"]][0])
    lean = 0.3 if case["kind"] == "batch" else 0.8
    head = _randn(_gen(seed, 6), embed.shape, s * math.sqrt(1.0 - lean * lean), embed.dtype)
    return head.add_(torch.roll(embed, 1, dims=0), alpha=s * lean)


def _cap(P, B):
    """Slots of a cache as a program allocates them: room for the prefix, the tree and the next cycles."""
    return (P + B + 128 + 63) // 64 * 64


def _caches(case, seed, tag, layers, cap):
    """Key and value caches of one request; random prefix (and random leftovers behind it)."""
    nkv, d, dt = MODELS[case["model"]][2], MODELS[case["model"]][3], DTYPES[case["dtype"]]
    g = _gen(seed, tag)
    return _randn(g, (layers, nkv, cap * d), 1.28, dt), _randn(g, (layers, nkv, cap * d), 1.28, dt)


def _tree(seed, B, vocab):
    """A spine of a third of the nodes with branches off earlier nodes; tokens: the first drafts of the spine continue the
    anchor (token + 1), the others are arbitrary and distinct."""
    rng = np.random.RandomState((int(seed) * 7919 + 13) % (1 << 31))
    spine = max(1, (B + 2) // 3)
    parent = np.array([-1] + [i - 1 if i < spine else rng.randint(0, i) for i in range(1, B)], dtype=np.int32)
    tokens = rng.permutation(vocab)[:B].astype(np.int32)
    for i in range(1, min(spine, ACCEPTED + 1)):
        tokens[i] = (tokens[0] + i) % vocab
    return tokens, parent, (np.arange(B) < spine).astype(np.uint8)


def _desc(case, layers):
    H, nh, nkv, d, F, V, base, eps, norm = MODELS[case["model"]]
    return goose.ModelDesc(layers, H, nh, d, F, V, base, eps, case["dtype"], nkv, norm, int(case["two_term"]))


def _requests(case, seed):
    """(B, P, tree seed) of every request of a case; requests of a batch differ in length and, by a few nodes, in size."""
    if case["kind"] != "batch":
        return [(case["B"], case["P"], seed)]
    return [(max(1, case["B"] - (r % 4 if case["B"] % 32 else 0)), max(1, case["P"] - (37 * r) % (case["P"] // 2 + 1)),
             int(seed) * 31 + r) for r in range(case["n"])]


def _pack_layers(ctx, case, seed, layers):
    lb = ctx.goose_packed_layer_bytes()
    packed = torch.zeros(layers * lb, dtype=torch.uint8, device=DEV)
    for l in range(layers):
        ctx.goose_pack_layer(_layer_weights(case, seed, l), packed[l * lb:(l + 1) * lb])
    return packed


def _pack_head(ctx, gain, head):
    packed = torch.zeros(ctx.goose_packed_lm_head_bytes(), dtype=torch.uint8, device=DEV)
    ctx.goose_pack_lm_head(gain, head, packed)
    return packed


def _head_rows(case, seed, head):
    """Final hidden rows of B nodes, each leaning towards one word of the head."""
    H, V = MODELS[case["model"]][0], MODELS[case["model"]][5]
    g = _gen(seed, 3)
    tokens = torch.randperm(V, generator=g, device=DEV)[:case["B"]]
    lean = head[tokens].float()
    return 0.15 * lean / lean.std() + _randn(g, (case["B"], H), 1.0, torch.float32), tokens.to(torch.int32)


def _i32(*shape, fill=0):
    return torch.full(shape, fill, dtype=torch.int32, device=DEV)


def prepare(case, seed):
    kind, B = case["kind"], case["B"]
    V, H = MODELS[case["model"]][5], MODELS[case["model"]][0]
    s = {"case": case}
    if kind == "layer":
        P, cap = case["P"], _cap(case["P"], B)
        ctx = s["ctx"] = GooseContext(_desc(case, 1), B, cap)
        s["layer"] = _pack_layers(ctx, case, seed, 1)
        s["embed"] = _embedding(case, seed)
        s["k"], s["v"] = _caches(case, seed, 4, 1, cap)
        tokens, parent, _ = _tree(seed, B, V)
        s["tokens"], parent = torch.from_numpy(tokens).to(DEV), torch.from_numpy(parent).to(DEV)
        s["mask"], depth, s["pos"] = torch.zeros(B * ((B + 63) // 64), dtype=torch.int64, device=DEV), _i32(B), _i32(B)
        ctx.goose_build_mask(parent, B, P, s["mask"], depth, s["pos"])
        s["x"] = torch.zeros((B, H), dtype=torch.float32, device=DEV)
    elif kind == "head":
        ctx = s["ctx"] = GooseContext(_desc(case, 1), B, 128)
        head = _randn(_gen(seed, 5), (V, H), 0.02 * math.sqrt(4096.0 / H), DTYPES[case["dtype"]])
        s["head"] = _pack_head(ctx, _final_gain(case, seed), head)
        s["x"], s["tokens"] = _head_rows(case, seed, head)
        s["argmax"], s["margin"] = _i32(B), torch.zeros(B, dtype=torch.float32, device=DEV)
        s["logits"] = torch.zeros((B, V), dtype=torch.float32, device=DEV)
        s["ids"], s["scores"] = _i32(V, HARVEST_K, fill=-1), torch.zeros((V, HARVEST_K), dtype=torch.float32, device=DEV)
    else:
        _prepare_steps(case, seed, s)
    torch.cuda.synchronize()
    return s


def _prepare_steps(case, seed, s):
    """A captured cycle over one request (goose_verify_step) or several (goose_verify_step_batched).  What changes from cycle
    to cycle -- tokens, parents, tags, cache lengths -- sits in one staging buffer that every pass copies in."""
    V = MODELS[case["model"]][5]
    reqs = _requests(case, seed)
    n, layers = len(reqs), STEP_LAYERS if case["kind"] == "step" else BATCH_LAYERS
    max_B, cap = max(b for b, _, _ in reqs), _cap(case["P"], case["B"])
    rows = sum((b + 31) // 32 * 32 for b, _, _ in reqs)
    ctx = s["ctx"] = GooseContext(_desc(case, layers), max_B, cap, rows if case["kind"] == "batch" else 0)
    s["layers"] = _pack_layers(ctx, case, seed, layers)
    s["embed"] = _embedding(case, seed)
    s["head"] = _pack_head(ctx, _final_gain(case, seed), _successor_head(case, seed, s["embed"]))
    kv = [_caches(case, seed, 1000 + r, layers, cap) for r in range(n)]
    s["k"], s["v"] = torch.stack([k for k, _ in kv]), torch.stack([v for _, v in kv])
    del kv
    host = np.zeros((n, 3, 128), dtype=np.int32)  # per request: tokens, parents, tags (bytes) + length in the last word
    for r, (b, p, ts) in enumerate(reqs):
        tokens, parent, spine = _tree(ts, b, V)
        host[r, 0, :b], host[r, 1, :b] = tokens, parent
        host[r, 2, :32].view(np.uint8)[:b] = spine
        host[r, 2, 127] = p
    s["staged"] = torch.from_numpy(host).to(DEV)
    s["live"] = torch.zeros_like(s["staged"])
    s["accept_len"], s["path"], s["bonus"] = _i32(n), _i32(n, 128, fill=-1), _i32(n)
    model = {"embed": s["embed"], "packed_layers": s["layers"], "packed_head": s["head"], "kcache": s["k"], "vcache": s["v"]}
    live = s["live"]
    if case["kind"] == "step":
        B = case["B"]
        s["argmax"] = _i32(B)
        s["logits"] = torch.zeros((B, V), dtype=torch.float32, device=DEV)
        s["margin"] = torch.zeros(B, dtype=torch.float32, device=DEV)
        io = {"tokens": live[0, 0], "parent": live[0, 1], "is_spine": live[0, 2].view(torch.uint8), "P": live[0, 2, 127:],
              "argmax": s["argmax"], "accept_len": s["accept_len"], "path": s["path"], "bonus": s["bonus"],
              "logits": s["logits"], "margin": s["margin"]}

        def call():
            ctx.goose_verify_step(model, io, B, cap - B)
    else:
        s["ids"] = _i32(n, V, HARVEST_K, fill=-1)
        s["scores"] = torch.zeros((n, V, HARVEST_K), dtype=torch.float32, device=DEV)
        s["argmax"] = _i32(rows)
        todo = [{"tokens": live[r, 0], "parent": live[r, 1], "is_spine": live[r, 2].view(torch.uint8), "B": b, "P_max": cap - b,
                 "kcache": s["k"][r], "vcache": s["v"][r], "P": live[r, 2, 127:], "accept_len": s["accept_len"][r:],
                 "path": s["path"][r], "bonus": s["bonus"][r:], "succ_ids": s["ids"][r], "succ_scores": s["scores"][r]}
                for r, (b, _, _) in enumerate(reqs)]

        def call():
            ctx.goose_verify_step_batched(model, todo, s["argmax"])
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        s["live"].copy_(s["staged"])
        call()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    s["graph"] = torch.cuda.CUDAGraph()
    with torch.cuda.graph(s["graph"]):
        call()
    torch.cuda.synchronize()


def run(s):
    case = s["case"]
    kind, B = case["kind"], case["B"]
    if kind == "layer":
        s["ctx"].goose_embed(s["embed"], s["tokens"], B, s["x"])
        s["ctx"].goose_verify_layer(s["layer"], s["x"], s["k"][0], s["v"][0], case["P"], B, s["mask"], s["pos"])
        return {"x": s["x"], "k": s["k"], "v": s["v"]}
    if kind == "head":
        s["ctx"].goose_lm_head_argmax(s["head"], s["x"], B, s["argmax"], s["logits"], s["margin"])
        s["ctx"].goose_harvest_topk(s["logits"], s["logits"].shape[1], s["tokens"], B, HARVEST_K, s["ids"], s["scores"])
        return {"argmax": s["argmax"], "logits": s["logits"], "margin": s["margin"], "ids": s["ids"], "scores": s["scores"]}
    s["live"].copy_(s["staged"])
    s["graph"].replay()
    out = {"argmax": s["argmax"], "accept_len": s["accept_len"], "path": s["path"], "bonus": s["bonus"],
           "length": s["live"], "k": s["k"], "v": s["v"]}
    out.update({"logits": s["logits"], "margin": s["margin"]} if kind == "step" else {"ids": s["ids"], "scores": s["scores"]})
    return out


# ---- what a pass cannot do without ------------------------------------------------------------------------
def work(case):
    H, nh, nkv, d, F, V = MODELS[case["model"]][:6]
    kind = case["kind"]
    es = 4 if case["dtype"] == "f32" else 2
    layers = {"layer": 1, "head": 0, "step": STEP_LAYERS, "batch": BATCH_LAYERS}[kind]
    params = nh * d * H * 2 + 2 * nkv * d * H + 3 * F * H
    nbytes = layers * params * es
    flops = 0.0
    for b, p, _ in _requests(case, 0):
        if kind != "head":
            nbytes += b * H * es + layers * 2 * nkv * d * (p + b) * es   # embedding rows; the prefix read, the tree's rows written
            flops += layers * (2.0 * b * params + 4.0 * b * nh * d * (p + b))
        if kind == "layer":
            nbytes += b * H * 4                                           # the residual rows handed back
        if kind != "layer":
            flops += 2.0 * b * V * H
        if kind in ("head", "step"):
            nbytes += b * V * 4 + (b * H * 4 if kind == "head" else 0)    # logits written, final rows read
        if kind in ("head", "batch"):
            nbytes += b * HARVEST_K * 8
    if kind != "layer":
        nbytes += V * H * es
    return {"bytes": float(nbytes), "flops": float(flops)}


def tolerance(case):
    # About four times the largest error against exact() over the listed and drawn cases (layer 4e-4, head 2e-4, batch 1.4e-3,
    # fp32 step 3e-7); "max" allows the odd cached row one more unit in its last place on top.
    if case["kind"] == "step":
        return {"rel": 2e-6, "max": 5e-5, "differ": 0.0}
    if case["kind"] == "head":
        return {"rel": 1e-3, "max": 1e-2, "differ": 1e-4}
    if case["kind"] == "batch":
        return {"rel": 5e-3, "max": 5e-2, "differ": 1e-3}
    return {"rel": 1.5e-3, "max": 2e-2}


# ---- the same in 64 bits, in plain torch -------------------------------------------------------------------
def _k_index(slots, d):
    """Element offset of (slot, column) inside one head's key cache, as goose.h lays it out (16-bit models)."""
    kk, c = (slots % 32).view(-1, 1), torch.arange(d, device=DEV).view(1, -1)
    i = ((kk // 4) % 4) * 8 + (kk // 16) * 4 + kk % 4
    return ((((slots // 32).view(-1, 1) * (d // 16)) + c // 16) * 64 + i + 32 * ((c // 8) % 2)) * 8 + c % 8


def _v_index(slots, d):
    kk, c = (slots % 32).view(-1, 1), torch.arange(d, device=DEV).view(1, -1)
    return ((((slots // 32).view(-1, 1) * (d // 32) + c // 32) * 2 + (kk // 8) % 2) * 64 + c % 32 + 32 * (kk // 16)) * 8 + kk % 8


def _index(case, slots, cap):
    """(key, value) element offsets of whole slots inside one head's cache."""
    d = MODELS[case["model"]][3]
    if case["dtype"] != "f32":
        return _k_index(slots, d), _v_index(slots, d)
    c = torch.arange(d, device=DEV).view(1, -1)
    return slots.view(-1, 1) * d + c, c * cap + slots.view(-1, 1)


def _norm(x, g, eps):
    return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + eps) * g.double()


def _layer64(case, w, x, reqs, trees, k, v, l, cap):
    """One decoder layer over the stacked rows x (fp64), every request on its own caches k, v (fp64, whole, updated)."""
    H, nh, nkv, d, F, V, base, eps, norm = MODELS[case["model"]]
    xn = _norm(x, w["g1"], eps)
    out = torch.empty((x.shape[0], nh * d), dtype=torch.float64, device=DEV)
    q_all, k_all, v_all = (xn @ w[n].double().t() for n in ("wq", "wk", "wv"))
    lo = 0
    for r, (b, p, _) in enumerate(reqs):
        parent = trees[r][1]
        anc = np.eye(b, dtype=bool)
        depth = np.zeros(b, dtype=np.int64)
        for i in range(1, b):
            anc[i] |= anc[parent[i]]
            depth[i] = depth[parent[i]] + 1
        q, kn, vn = (t[lo:lo + b].view(b, -1, d).transpose(0, 1).contiguous() for t in (q_all, k_all, v_all))
        if norm:
            q, kn = _norm(q, w["gq"], eps), _norm(kn, w["gk"], eps)
        ang = torch.from_numpy(p + depth).to(DEV).double().view(-1, 1) * base ** (
            -2.0 * torch.arange(d // 2, device=DEV).double() / d)
        cos, sin = torch.cos(ang), torch.sin(ang)

        def rot(t):
            a, c = t[..., :d // 2], t[..., d // 2:]
            return torch.cat([a * cos - c * sin, c * cos + a * sin], dim=-1)

        q, kn = rot(q), rot(kn)
        ki, vi = _index(case, torch.arange(p + b, device=DEV), cap)
        k[r, l][:, ki[p:]], v[r, l][:, vi[p:]] = kn, vn
        see = torch.cat([torch.ones((b, p), dtype=torch.bool, device=DEV), torch.from_numpy(anc).to(DEV)], dim=1)
        for j in range(nkv):
            kk, vv = k[r, l, j][ki], v[r, l, j][vi]
            for h in range(j * (nh // nkv), (j + 1) * (nh // nkv)):
                a = (q[h] @ kk.t()) / math.sqrt(d)
                a = torch.softmax(a.masked_fill(~see, float("-inf")), dim=-1)
                out[lo:lo + b, h * d:(h + 1) * d] = a @ vv
        lo += b
    x = x + out @ w["wo"].double().t()
    xn = _norm(x, w["g2"], eps)
    gate, up = xn @ w["wg"].double().t(), xn @ w["wu"].double().t()
    return x + (gate * torch.sigmoid(gate) * up) @ w["wd"].double().t()


def _logits64(case, x, gain, head):
    xn = _norm(x, gain, MODELS[case["model"]][7])
    return torch.cat([xn @ c.double().t() for c in head.split(16384)], dim=1)


def _top(logits, tokens, scores):
    top = torch.topk(torch.softmax(logits, dim=-1), HARVEST_K, dim=-1).values
    for i, t in enumerate(tokens):  # (a later node with the same token wins)
        scores[int(t)] = top[i]


def exact(case, seed):
    H, V, kind = MODELS[case["model"]][0], MODELS[case["model"]][5], case["kind"]
    if kind == "head":
        head = _randn(_gen(seed, 5), (V, H), 0.02 * math.sqrt(4096.0 / H), DTYPES[case["dtype"]])
        x, tokens = _head_rows(case, seed, head)
        logits = _logits64(case, x.double(), _final_gain(case, seed), head)
        two = torch.topk(logits, 2, dim=-1).values
        scores = torch.zeros((V, HARVEST_K), dtype=torch.float64, device=DEV)
        _top(logits, tokens.cpu(), scores)
        return {"argmax": None, "logits": logits, "margin": two[:, 0] - two[:, 1], "ids": None, "scores": scores}
    reqs = _requests(case, seed)
    trees = [_tree(ts, b, V) for b, _, ts in reqs]
    layers = {"layer": 1, "step": STEP_LAYERS, "batch": BATCH_LAYERS}[kind]
    cap = _cap(case["P"], case["B"])
    kv = [_caches(case, seed, 4 if kind == "layer" else 1000 + r, layers, cap) for r in range(len(reqs))]
    k, v = torch.stack([a for a, _ in kv]).double(), torch.stack([a for _, a in kv]).double()
    del kv
    embed = _embedding(case, seed)
    x = embed[torch.from_numpy(np.concatenate([t for t, _, _ in trees])).to(DEV).long()].double()
    for l in range(layers):
        x = _layer64(case, _layer_weights(case, seed, l), x, reqs, trees, k, v, l, cap)
    if kind == "layer":
        return {"x": x, "k": k[0], "v": v[0]}
    head, gain = _successor_head(case, seed, embed), _final_gain(case, seed)
    out = {"argmax": None, "accept_len": None, "path": None, "bonus": None, "length": None}
    scores = torch.zeros((len(reqs), V, HARVEST_K), dtype=torch.float64, device=DEV) if kind == "batch" else None
    lo = 0
    for r, (b, p, _) in enumerate(reqs):
        tokens, parent, spine = trees[r]
        logits = _logits64(case, x[lo:lo + b], gain, head)
        lo += b
        best = torch.topk(logits, 2, dim=-1)
        word = best.indices[:, 0].cpu().numpy()
        path = [0]
        while True:  # the accepted path: spine child first, then the lowest index
            hit = [i for i in range(1, b) if parent[i] == path[-1] and tokens[i] == word[path[-1]]]
            if not hit:
                break
            path.append(min(hit, key=lambda i: (not spine[i], i)))
        ki, vi = _index(case, torch.arange(cap, device=DEV), cap)
        src, dst = [p + i for i in path], list(range(p, p + len(path)))
        k[r][..., ki[dst]], v[r][..., vi[dst]] = k[r][..., ki[src]], v[r][..., vi[src]]
        if kind == "batch":
            _top(logits, tokens, scores[r])
    out.update({"k": k, "v": v})
    out.update({"logits": logits, "margin": best.values[:, 0] - best.values[:, 1]} if kind == "step"
               else {"ids": None, "scores": scores})
    return out
