"""The calls whose speed counts: the stages of a semantic-parallel MoE layer through `SemMoE`, and two whole layers.

Shapes are those of `workloads.CONFIGS`; token counts run from a few tokens of decode to a prefill batch.  A case names
one operation (`op`) and plain sizes:

  layer   route -> reshuffle -> dispatch -> expert_ffn (all ranks) -> combine
  route   router GEMM and top-k selection, the logits not asked for
  index   reshuffle and dispatch_index: everything that is decided about tokens and pairs before a row moves
  rows    dispatch_rows and combine: the row moves of a layer, without the FFN between them
  ffn     grouped SwiGLU FFN of one rank's experts (rank >= 0) or of all of them (rank = -1)
  shared  FFN of the shared expert on one rank's shard of tokens
"""
import math

import torch

import paper_2503_04398_amd as S

DEV = "cuda:0"

# hidden width, experts, experts per token, FFN width, ranks, routing classes, scoring
SHAPES = {
    "tiny": dict(d=512, E=16, k=2, F=1024, D=4, C=4, dtype="fp32", score="softmax", renorm=False, n_group=1, topk_group=1),
    "qwen3_30b": dict(d=2048, E=128, k=8, F=768, D=8, C=16, dtype="bf16", score="softmax", renorm=True, n_group=1, topk_group=1),
    "qwen3_235b": dict(d=4096, E=128, k=8, F=1536, D=8, C=16, dtype="bf16", score="softmax", renorm=True, n_group=1, topk_group=1),
    "gpt_oss_120b": dict(d=2880, E=128, k=4, F=2880, D=16, C=32, dtype="bf16", score="softmax", renorm=True, n_group=1, topk_group=1),
    "deepseek_v3": dict(d=7168, E=256, k=8, F=2048, D=32, C=32, dtype="bf16", score="sigmoid", renorm=True, n_group=8, topk_group=4),
}


def listed():
    def case(name, op, shape, **kw):
        return dict(name=name, op=op, **SHAPES[shape], **kw)

    return [
        # a small fp32 layer, every launch of it short: what a test system or a small model runs
        case("layer_tiny_fp32", "layer", "tiny", T=256),
        # one decode step of a few requests through a whole layer on one GPU: streams nearly all experts once
        case("layer_decode", "layer", "qwen3_235b", T=64),
        # the gate of a decode step
        case("route_decode", "route", "qwen3_235b", T=256),
        # the gate of a prefill batch: softmax, and group-limited sigmoid over twice the experts
        case("route_softmax_prefill", "route", "qwen3_30b", T=8192),
        case("route_sigmoid_prefill", "route", "deepseek_v3", T=16384),
        # the integer half of scheduling a prefill batch
        case("index_prefill", "index", "deepseek_v3", T=16384),
        # the rows of that batch into expert order and back
        case("rows_prefill", "rows", "deepseek_v3", T=16384),
        # experts of the most loaded rank under an affinity placement (prefill)
        case("ffn_prefill_narrow", "ffn", "qwen3_30b", T=8192, rank=0, rows=20865, skew=0.3),
        case("ffn_prefill_wide", "ffn", "gpt_oss_120b", T=32768, rank=0, rows=9826, skew=0.1),
        # experts of one rank in a decode step
        case("ffn_decode", "ffn", "qwen3_235b", T=256, rank=0, rows=263, skew=0.2),
        # a chunk of prefill with all experts on one GPU, a ragged token count: neither few rows per expert nor many
        case("ffn_chunk", "ffn", "qwen3_30b", T=1000, rank=-1, rows=8000, skew=0.5),
        # the shared expert on one rank's shard of the prefill batch
        case("shared_shard", "shared", "deepseek_v3", T=16384, n_tokens=512),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["layer", "route", "route", "index", "rows", "ffn", "ffn", "ffn", "shared"])
    shape = rng.choice(["qwen3_30b", "qwen3_235b", "gpt_oss_120b", "deepseek_v3"])
    c = dict(op=op, **SHAPES[shape])
    if op == "layer":
        c = dict(op=op, **SHAPES[rng.choice(["tiny", "qwen3_30b", "qwen3_235b"])])
        c["T"] = _log_int(rng, 1, 64 if c["d"] == 4096 else 500)
        if c["dtype"] == "fp32":
            c["d"], c["F"] = 8 * _log_int(rng, 32, 128), 8 * _log_int(rng, 32, 160)
    elif op == "route":
        c["T"] = _log_int(rng, 16, 16384)
    elif op == "index":
        c["T"] = _log_int(rng, 16, 32768)
    elif op == "rows":
        c["T"] = _log_int(rng, 16, 16384)
    elif op == "shared":
        c.update(SHAPES[rng.choice(["qwen3_30b", "qwen3_235b", "deepseek_v3"])])
        c["n_tokens"] = _log_int(rng, 16, 2048)
        c["T"] = 8 * c["n_tokens"]
    else:
        if rng.random() < 0.25:  # a width that is no multiple of the tiles
            c["d"], c["F"] = 8 * rng.randrange(128, 360), 8 * rng.randrange(64, 240)
        m = c["E"] // c["D"]
        c["rank"] = rng.choice([0, c["D"] - 1]) if c["E"] * c["F"] * c["d"] > 5e8 else rng.choice([-1, 0, c["D"] - 1])
        groups = m if c["rank"] >= 0 else c["E"]
        most = min(1200 if c["rank"] >= 0 else 200, int(7e10 / (groups * c["d"] * c["F"])))
        c["rows"] = groups * _log_int(rng, 2, most) + rng.randrange(groups)
        c["skew"] = rng.choice([0.1, 0.3, 1.0])
        c["T"] = -(-c["rows"] // c["k"]) * (rng.choice([2, c["D"] // 2]) if c["rank"] >= 0 else 1)
    return c


# ------------------------------------------------------------------------------------------------------ inputs
def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _act(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _randn(g, shape, std, dtype):
    return torch.empty(shape, dtype=dtype, device=DEV).normal_(0.0, std, generator=g)


def _config(case, **kw):
    T, D = case["T"], case["D"]
    return S.Config(T=T, d=case["d"], E=case["E"], k=case["k"], F=case["F"], D=D, dtype=case["dtype"], score=case["score"],
                    renorm=case["renorm"], n_group=case["n_group"], topk_group=case["topk_group"],
                    routed_scale=2.5 if case["score"] == "sigmoid" else 1.0, cap=-(-T // D), num_classes=case["C"], **kw)


def _i32(*shape):
    return torch.empty(shape, dtype=torch.int32, device=DEV)


def _classes(case, g):
    """Tokens belong to latent classes (a few of them popular), a class leans on a cluster of experts, the ids of which are
    scattered: token_class[T], class_bias[C,E] and the order in which a placement by affinity puts the experts."""
    T, E, C, m = case["T"], case["E"], case["C"], case["E"] // case["D"]
    p = torch.arange(1, C + 1, device=DEV, dtype=torch.float32).pow(-1.1 if case["score"] == "softmax" else 0.0)
    cls = torch.multinomial(p, T, replacement=True, generator=g).to(torch.int32)
    order = torch.randperm(E, device=DEV, generator=g)
    at = (torch.arange(C, device=DEV)[:, None] * max(E // C, 1) + torch.arange(m, device=DEV)) % E
    bias = torch.zeros(C, E, device=DEV).scatter_(1, order[at], 1.5)
    return cls, bias, order


def _placement(case, order):
    E, m = case["E"], case["E"] // case["D"]
    rank = torch.empty(E, dtype=torch.int64, device=DEV)
    rank[order] = torch.arange(E, device=DEV) // m
    of_phys = torch.argsort(rank * E + torch.arange(E, device=DEV))  # rank by rank, ascending ids inside a rank
    phys = torch.empty_like(of_phys)
    phys[of_phys] = torch.arange(E, device=DEV)
    return rank.to(torch.int32), phys.to(torch.int32), of_phys.to(torch.int32)


def _router(s, case, g):
    T, d, E, k = case["T"], case["d"], case["E"], case["k"]
    s["X"] = _randn(g, (T, d), 1.0, _act(case))
    s["W_r"] = _randn(g, (E, d), 0.02, _act(case))
    s["cls"], s["class_bias"], s["order"] = _classes(case, g)
    s["sel_bias"] = _randn(g, (E,), 0.05, torch.float32) if case["score"] == "sigmoid" else None
    s["ids"], s["w"] = _i32(T, k), torch.empty(T, k, device=DEV)


def _index_buffers(s, case):
    T, E, k, D = case["T"], case["E"], case["k"], case["D"]
    s.update(token_rank=_i32(T), shf=_i32(T), inv_shf=_i32(T), rank_count=_i32(D), slot_of_pair=_i32(T * k),
             pair_of_slot=_i32(T * k), expert_offsets=_i32(E + 1), rank_offsets=_i32(D + 1), send_matrix=_i32(D, D),
             remote_pairs=torch.empty(1, dtype=torch.int64, device=DEV))


def prepare(case, seed):
    g = _gen(seed)
    op, T, d, E, k, F, D = (case[n] for n in ("op", "T", "d", "E", "k", "F", "D"))
    P, m, act = T * k, E // D, _act(case)
    s = {"op": op, "rank": case.get("rank", -1), "m": S.SemMoE(_config(case), device=DEV)}
    if op in ("layer", "route"):
        _router(s, case, g)
    if op == "layer":
        s["e2r"], s["phys"], s["of_phys"] = _placement(case, s["order"])
        _index_buffers(s, case)
        s["W_gu"], s["W_down"] = _randn(g, (E, 2 * F, d), 0.02, act), _randn(g, (E, d, F), 0.02, act)
        s["X_perm"], s["Y"] = (torch.empty(P, d, dtype=act, device=DEV) for _ in range(2))
        s["Out"] = torch.empty(T, d, dtype=act, device=DEV)
    elif op == "index":
        cls, bias, order = _classes(case, g)
        scores = _randn(g, (T, E), 1.3, torch.float32) + bias[cls.long()]
        s["ids"] = scores.topk(k, dim=1).indices.to(torch.int32).contiguous()
        s["e2r"], s["phys"], _ = _placement(case, order)
        _index_buffers(s, case)
    elif op == "rows":
        s["X"], s["Y"] = _randn(g, (T, d), 1.0, act), _randn(g, (P, d), 0.2, act)
        s["slot_of_pair"] = torch.randperm(P, device=DEV, generator=g).to(torch.int32)
        s["w"] = torch.rand(T, k, device=DEV, generator=g).softmax(1).contiguous()
        s["X_perm"], s["Out"] = torch.empty(P, d, dtype=act, device=DEV), torch.empty(T, d, dtype=act, device=DEV)
    elif op == "ffn":
        rank, rows = case["rank"], case["rows"]
        lo, n = (rank * m, m) if rank >= 0 else (0, E)
        counts = torch.zeros(E, dtype=torch.int64, device=DEV)
        p = _randn(g, (E,), case["skew"], torch.float32).exp()
        counts[lo:lo + n] = torch.bincount(torch.multinomial(p[lo:lo + n], rows, replacement=True, generator=g), minlength=n)
        if n < E:  # the pairs of the other ranks lie before and after this rank's
            p[lo:lo + n] = 0
            counts += torch.bincount(torch.multinomial(p, P - rows, replacement=True, generator=g), minlength=E)
        s["expert_offsets"] = torch.cat([counts.new_zeros(1), counts.cumsum(0)]).to(torch.int32)
        # a rank's program holds the weights of its own experts
        s["of_phys"] = (torch.randperm(n, device=DEV, generator=g)).to(torch.int32).repeat(E // n).contiguous()
        s["W_gu"], s["W_down"] = _randn(g, (n, 2 * F, d), 0.02, act), _randn(g, (n, d, F), 0.02, act)
        s["X_perm"] = _randn(g, (max(P, int(counts.sum())), d), 1.0, act)
        s["Y"] = torch.zeros_like(s["X_perm"])
    elif op == "shared":
        n = case["n_tokens"]
        s["X"] = _randn(g, (n, d), 1.0, act)
        s["W_gu"], s["W_down"] = _randn(g, (2 * F, d), 0.02, act), _randn(g, (d, F), 0.02, act)
        s["Y"] = torch.empty(n, d, dtype=act, device=DEV)
    return s


# --------------------------------------------------------------------------------------------------- the calls
def run(s):
    m, op = s["m"], s["op"]
    if op in ("layer", "route"):
        m.route(s["X"], s["W_r"], s["ids"], s["w"], token_class=s["cls"], class_bias=s["class_bias"], sel_bias=s["sel_bias"])
        if op == "route":
            return {"ids": s["ids"], "w": s["w"]}
    if op == "layer":
        m.reshuffle(s["ids"], s["e2r"], s["token_rank"], s["shf"], s["inv_shf"], s["rank_count"])
        m.dispatch(s["X"], s["ids"], s["token_rank"], s["shf"], s["phys"], s["X_perm"], s["slot_of_pair"], s["pair_of_slot"],
                   s["expert_offsets"], s["rank_offsets"], s["send_matrix"], s["remote_pairs"])
        m.expert_ffn(-1, s["X_perm"], s["expert_offsets"], s["of_phys"], s["W_gu"], s["W_down"], s["Y"])
        m.combine(s["Y"], s["slot_of_pair"], s["w"], s["Out"])
        return {"ids": s["ids"], "w": s["w"], "out": s["Out"]}
    if op == "index":
        m.reshuffle(s["ids"], s["e2r"], s["token_rank"], s["shf"], s["inv_shf"], s["rank_count"])
        m.dispatch_index(s["ids"], s["token_rank"], s["shf"], s["phys"], s["slot_of_pair"], s["pair_of_slot"],
                         s["expert_offsets"], s["rank_offsets"], s["send_matrix"], s["remote_pairs"])
        return {n: s[n] for n in ("token_rank", "shf", "inv_shf", "rank_count", "slot_of_pair", "pair_of_slot",
                                  "expert_offsets", "rank_offsets", "send_matrix", "remote_pairs")}
    if op == "rows":
        m.dispatch_rows(s["X"], s["slot_of_pair"], s["X_perm"])
        m.combine(s["Y"], s["slot_of_pair"], s["w"], s["Out"])
        return {"X_perm": s["X_perm"], "out": s["Out"]}
    if op == "ffn":
        m.expert_ffn(s["rank"], s["X_perm"], s["expert_offsets"], s["of_phys"], s["W_gu"], s["W_down"], s["Y"])
        return {"y": s["Y"]}
    m.shared_ffn(s["X"], s["X"].shape[0], s["W_gu"], s["W_down"], s["Y"])
    return {"y": s["Y"]}


def work(case):
    T, d, E, k, F, D = (case[n] for n in ("T", "d", "E", "k", "F", "D"))
    b, P = (2 if case["dtype"] == "bf16" else 4), T * k

    def ffn(rows, groups):
        used = groups * (1.0 - (1.0 - 1.0 / groups) ** rows)  # experts that get a row
        return {"bytes": 2 * rows * d * b + used * 3 * F * d * b, "flops": 6 * rows * d * F}

    route = {"bytes": T * d * b + E * d * b + P * 8 + T * 4 + case["C"] * E * 4, "flops": 2 * T * d * E}
    index = {"bytes": 4 * (P + 3 * T + 2 * P), "flops": 0}
    rows = {"bytes": 2 * (T + P) * d * b + P * 8, "flops": 2 * P * d}
    if case["op"] == "layer":
        f = ffn(P, E)  # X read once, the output written once; what lies between the stages is not counted
        return {"bytes": route["bytes"] + T * d * b + f["bytes"] - 2 * P * d * b, "flops": route["flops"] + f["flops"] + 2 * P * d}
    if case["op"] == "ffn":
        return ffn(case["rows"], E // D if case["rank"] >= 0 else E)
    if case["op"] == "shared":
        return ffn(case["n_tokens"], 1)
    return {"route": route, "index": index, "rows": rows}[case["op"]]


def tolerance(case):
    # whole numbers of the scheduling half follow from whole numbers
    if case["op"] == "index":
        return "exact"
    # fp32 sums; ids of two experts whose logits agree to the last bits may change places
    if case["op"] == "route":
        return {"rel": 1e-4, "max": 0.5, "differ": 1e-3 if case["T"] >= 1024 else 0.01}
    if case["op"] == "layer" and case["dtype"] == "fp32":
        return {"rel": 1e-5, "max": 1e-4, "differ": 0.01}
    if case["op"] == "rows":
        return {"rel": 2e-3, "max": 1e-2}  # one rounding to bf16
    return {"rel": 8e-3, "max": 6e-2, "differ": 0.01}  # bf16 hidden activations and results


# ------------------------------------------------------------------------------------------------ in 64 bits
def _swiglu(x, w_gu, w_down):
    F = w_down.shape[1]
    gate, up = x @ w_gu[:F].double().t(), x @ w_gu[F:].double().t()
    return (gate * torch.sigmoid(gate) * up) @ w_down.double().t()


def _select(case, s):
    E, k = case["E"], case["k"]
    logits = s["X"].double() @ s["W_r"].double().t() + s["class_bias"].double()[s["cls"].long()]
    if case["score"] == "softmax":
        ids = logits.topk(k, dim=1).indices
        w = logits.softmax(1).gather(1, ids)
        return ids, (w / w.sum(1, keepdim=True) if case["renorm"] else w)
    sig = torch.sigmoid(logits)
    pick, ng = sig + s["sel_bias"].double(), case["n_group"]
    best = pick.view(-1, ng, E // ng).topk(2, dim=2).values.sum(2).topk(case["topk_group"], dim=1).indices
    keep = torch.zeros(pick.shape[0], ng, dtype=torch.bool, device=DEV).scatter_(1, best, True)
    ids = pick.masked_fill(~keep.repeat_interleave(E // ng, 1), float("-inf")).topk(k, dim=1).indices
    w = sig.gather(1, ids)
    return ids, w / w.sum(1, keepdim=True) * 2.5


def exact(case, seed):
    op, k = case["op"], case["k"]
    if op == "index":
        return None
    s = prepare(case, seed)
    if op in ("layer", "route"):
        ids, w = _select(case, s)
        if op == "route":
            return {"ids": None, "w": w}
        out = torch.zeros(case["T"], case["d"], dtype=torch.float64, device=DEV)
        for e in ids.unique().tolist():
            tok, j = (ids == e).nonzero(as_tuple=True)
            out.index_add_(0, tok, w[tok, j, None] * _swiglu(s["X"][tok].double(), s["W_gu"][e], s["W_down"][e]))
        return {"ids": None, "w": w, "out": out}
    if op == "rows":
        out = torch.zeros(s["Out"].shape, dtype=torch.float64, device=DEV)
        slots = s["slot_of_pair"].view(-1, k).long()
        for j in range(k):
            out += s["w"][:, j, None].double() * s["Y"][slots[:, j]].double()
        return {"X_perm": None, "out": out}
    if op == "shared":
        return {"y": _swiglu(s["X"].double(), s["W_gu"], s["W_down"])}
    y = torch.zeros(s["Y"].shape, dtype=torch.float64, device=DEV)
    off, m = s["expert_offsets"].tolist(), case["E"] // case["D"]
    for q in range(case["rank"] * m, case["rank"] * m + m) if case["rank"] >= 0 else range(case["E"]):
        if off[q + 1] > off[q]:
            e = int(s["of_phys"][q])
            y[off[q]:off[q + 1]] = _swiglu(s["X_perm"][off[q]:off[q + 1]].double(), s["W_gu"][e], s["W_down"][e])
    return {"y": y}
