"""The calls whose time on one MI355X stands for the use of this library.

The path is one MoE layer of a decode step: `base_decode_layer` (or its
staged calls) on a batch of one token per active sequence, under an expert
budget.  Beside it stand the layer stack of a decode step, the predictor's
calibration statistics and the packing of a loaded layer's experts.  Shapes
are those of the models in `workloads` (Qwen3-30B-A3B, OLMoE, Mixtral,
DeepSeek-V2-Lite, Qwen1.5-MoE) and the distributions follow the same recipe,
drawn on the GPU: RMS-normalised rows (half of them around four centres where
the batch is clustered), a Zipf-biased router, experts of std 1/sqrt(fan_in).
"""
import math

import torch

from paper_2609_36222_amd import binding as bd

DECODE = dict(kind="decode", dtype="bf16", layers=1, staged=False, packed=True, norm_topk=1,
              rule=0, flags=0, residual=False, clustered=False, n_shared=0, shared_gate=False)
QWEN3 = dict(DECODE, d=2048, E=128, K=8, I=768)


def listed():
    return [
        # the fp32 layer of the parity tests and of small experiments: every
        # launch is tiny, the call is its latency
        dict(DECODE, name="tiny_fp32_b8", dtype="f32", packed=False, d=256, E=16, K=2, I=512, B=8,
             budget=6),
        # one sequence being served: the smallest decode step
        dict(QWEN3, name="qwen3_b1", B=1, budget=10, residual=True),
        # the method's own operating point: batch 16 with ten kept experts
        dict(QWEN3, name="qwen3_b16", B=16, budget=10),
        # a small batch on a model of fewer, wider experts
        dict(DECODE, name="olmoe_b32", d=2048, E=64, K=8, I=1024, B=32, budget=16),
        # a serving engine that runs its own schedule between the calls
        dict(QWEN3, name="qwen3_b64_staged", B=64, budget=32, staged=True),
        # the headline layer: a large, half clustered batch
        dict(QWEN3, name="qwen3_b256", B=256, budget=32, clustered=True),
        # the largest batch with every expert kept (dense serving)
        dict(QWEN3, name="qwen3_b1024_all", B=1024, budget=128),
        # few, large experts
        dict(DECODE, name="mixtral_b128", d=4096, E=8, K=2, I=14336, B=128, budget=4),
        # a ragged batch on weights as the checkpoint holds them (row-major),
        # raw softmax weights, gated shared experts, renormalised gates
        dict(DECODE, name="qwen15_b61_rowmajor", d=2048, E=60, K=4, I=1408, B=61, budget=16,
             packed=False, norm_topk=0, flags=1, n_shared=4, shared_gate=True),
        # a decode step's layer stack: eight layers, own weights and inputs,
        # the residual stream added
        dict(QWEN3, name="qwen3_stack8_b128", B=128, budget=24, layers=8, residual=True),
        # calibration: statistics of two batches of tokens from zero
        dict(kind="calib", name="calib_olmoe", d=2048, E=64, K=8, I=1024, B=1024, batches=2),
        # load time: one layer's experts into the packed layout
        dict(kind="pack", name="pack_olmoe", d=2048, E=64, I=1024),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


# bounds that keep a drawn case below the largest listed one
_KEPT_BYTES, _ALL_BYTES, _PAIR_WORK = 1.2e9, 2.5e9, 1.2e10


def draw(rng):
    kind = rng.choice(["decode"] * 7 + ["f32", "calib", "pack"])
    if kind == "f32":
        E = _log_int(rng, 4, 32)
        return dict(DECODE, dtype="f32", packed=False, d=256 * rng.randint(1, 2), E=E,
                    K=rng.randint(1, min(4, E)), I=64 * rng.randint(1, 8), B=_log_int(rng, 1, 64),
                    budget=rng.randint(1, E), flags=rng.choice([0, 0, 1, 2, 3]),
                    norm_topk=rng.randint(0, 1))
    if kind == "pack":
        d, I = 256 * _log_int(rng, 2, 16), 64 * _log_int(rng, 2, 44)
        return dict(kind="pack", d=d, I=I, E=max(1, min(_log_int(rng, 4, 256), int(8e8 / (6 * d * I)))))
    if kind == "calib":
        E = _log_int(rng, 8, 64)
        return dict(kind="calib", d=256 * _log_int(rng, 1, 8), E=E, K=rng.randint(1, min(8, E)),
                    I=64 * _log_int(rng, 1, 16), B=_log_int(rng, 16, 1024), batches=rng.randint(1, 2))
    E, d = _log_int(rng, 8, 256), 256 * _log_int(rng, 2, 16)
    K, B, budget = rng.randint(1, min(10, E)), _log_int(rng, 1, 1024), _log_int(rng, 1, E)
    layers = rng.choice([1, 1, 1, 1, 3])
    ns = rng.choice([0, 0, 0, 1, 2, 4])
    I = 64 * _log_int(rng, 1, 224)
    most = min(_ALL_BYTES / (6 * d * (E + ns)), _KEPT_BYTES / (6 * d * (min(budget, E) + ns)),
               _PAIR_WORK / (B * (K + ns) * d)) / layers
    return dict(DECODE, d=d, E=E, K=K, B=B, budget=budget, layers=layers, n_shared=ns,
                I=max(64, min(I, int(most) // 64 * 64)), shared_gate=bool(ns) and rng.random() < 0.5,
                packed=rng.random() < 0.7, staged=layers == 1 and rng.random() < 0.2,
                clustered=rng.random() < 0.3, residual=rng.random() < 0.5,
                norm_topk=rng.randint(0, 1), flags=rng.choice([0, 0, 0, 1, 2]),
                rule=rng.choice([0, 0, 0, 0, 1, 2, 3, 4]))


# ------------------------------------------------------------------ inputs --
def _gen(seed, layer, stream):
    g = torch.Generator(device="cuda")
    g.manual_seed((seed * 1009 + layer) * 16 + stream)
    return g


def _normal(g, shape, std, dtype=torch.float32):
    return torch.randn(shape, generator=g, device="cuda", dtype=dtype).mul_(std)


def _dtype(case):
    return torch.float32 if case.get("dtype") == "f32" else torch.bfloat16


def _tokens(case, seed, layer, stream=0):
    B, d, g = case["B"], case["d"], _gen(seed, layer, stream)
    z = _normal(g, (B, d), 1.0)
    if case.get("clustered") and B >= 2:
        nc = B // 2
        centres = _normal(g, (4, d), 1.0)
        pick = torch.randint(0, 4, (nc,), generator=g, device="cuda")
        z[:nc] = centres[pick] + 0.1 * z[:nc]
        z = z[torch.randperm(B, generator=g, device="cuda")]
    if _dtype(case) == torch.float32:
        return z
    return (z / (z.square().mean(1, keepdim=True) + 1e-6).sqrt()).to(torch.bfloat16)


def _router(case, seed, layer):
    E, d, g = case["E"], case["d"], _gen(seed, layer, 1)
    if _dtype(case) == torch.float32:
        return _normal(g, (E, d), 0.02), _normal(g, (E,), 0.5)
    rank = torch.randperm(E, generator=g, device="cuda").double() + 1.0
    p = rank ** -1.1
    return _normal(g, (E, d), 0.075), (p / p.sum()).log().float()


def _predictor(case, seed, layer):
    g, d = _gen(seed, layer, 2), case["d"]
    a = _normal(g, (case["E"], d), 0.3)
    return a, math.log(0.18 * d) + _normal(g, (case["E"],), 0.25)


def _experts(case, seed, layer, E, stream=3):
    d, I, dt, g = case["d"], case["I"], _dtype(case), _gen(seed, layer, stream)
    return _normal(g, (E, 2 * I, d), d ** -0.5, dt), _normal(g, (E, d, I), I ** -0.5, dt)


def _shared(case, seed, layer):
    if not case["n_shared"]:
        return None
    w13, w2 = _experts(case, seed, layer, case["n_shared"], 4)
    gate = _normal(_gen(seed, layer, 5), (case["d"],), case["d"] ** -0.5)
    return w13, w2, (gate if case["shared_gate"] else None)


def prepare(case, seed):
    if case["kind"] == "pack":
        w13, w2 = _experts(case, seed, 0, case["E"])
        layer = bd.Layer(torch.empty(case["E"], case["d"], device="cuda"), None, None, None, w13, w2)
        return dict(case=case, layer=layer, desc=layer.desc(1), out=(torch.empty_like(w13),
                                                                     torch.empty_like(w2)))
    if case["kind"] == "calib":
        w13, w2 = _experts(case, seed, 0, case["E"])
        layer = bd.Layer(*_router(case, seed, 0), None, None, w13, w2)
        layer = bd.packed_layer(layer, case["K"])
        z = [_tokens(case, seed, 0, 6 + b) for b in range(case["batches"])]
        desc = layer.desc(case["K"])
        ws = bd.calib_accumulate(desc, z[0], case["B"], bd.calib_stats(desc))
        return dict(case=case, layer=layer, desc=desc, z=z, ws=ws)
    B, d, E, K, dt = case["B"], case["d"], case["E"], case["K"], _dtype(case)
    bc = min(case["budget"], E)
    steps, ws = [], None
    for l in range(case["layers"]):
        layer = bd.Layer(*_router(case, seed, l), *_predictor(case, seed, l),
                         *_experts(case, seed, l, E), case["norm_topk"], score_rule=case["rule"],
                         shared=_shared(case, seed, l))
        if case["packed"]:
            layer = bd.packed_layer(layer, K)
        desc = layer.desc(K)
        if ws is None:
            ws = torch.empty(bd.base_workspace_bytes(desc, B, case["budget"]), dtype=torch.uint8,
                             device="cuda")
        steps.append(dict(layer=layer, desc=desc, x=_tokens(case, seed, l),
                          residual=_tokens(case, seed, l, 7) if case["residual"] else None,
                          y=torch.empty(B, d, dtype=dt, device="cuda")))
    st = dict(case=case, steps=steps, ws=ws)
    if case["staged"]:
        def f32(*s):
            return torch.empty(s, dtype=torch.float32, device="cuda")

        def i32(*s):
            return torch.empty(s, dtype=torch.int32, device="cuda")
        st["plan"] = dict(logits=f32(B, E), ids=i32(B, K), w=f32(B, K), cost=f32(B, K),
                          scores=f32(E), counts=i32(E), sel=i32(bc), n_sel=i32(1), slot=i32(E))
    return st


# --------------------------------------------------------------- one pass --
def _up256(v):
    return (v + 255) // 256 * 256


def _stats_views(stats, E, d):
    """The statistics buffer's arrays, in the order include/base.h gives."""
    o1 = _up256(E * 32)
    o2 = o1 + _up256(E * d * 8)
    o3 = o2 + _up256(E * d * 8)
    return dict(head=stats[:E * 32].view(torch.float64).view(E, 4),
                sz=stats[o1:o1 + E * d * 8].view(torch.float64).view(E, d),
                q=stats[o2:o2 + E * d * 8].view(torch.float64).view(E, d),
                G=stats[o3:o3 + E * d * d * 4].view(torch.float32).view(E, d, d))


def run(st):
    case = st["case"]
    if case["kind"] == "pack":
        bd.base_pack_experts(st["desc"], *st["out"])
        return st["out"]
    if case["kind"] == "calib":
        stats = bd.calib_stats(st["desc"])
        for z in st["z"]:
            bd.calib_accumulate(st["desc"], z, case["B"], stats, st["ws"])
        return _stats_views(stats, case["E"], case["d"])
    if not case["staged"]:
        for s in st["steps"]:
            bd.base_decode_layer(s["desc"], s["x"], case["B"], case["budget"], case["flags"],
                                 s["residual"], s["y"], st["ws"])
        return [s["y"] for s in st["steps"]]
    s, p, B = st["steps"][0], st["plan"], case["B"]
    bd.base_route(s["desc"], s["x"], B, p["logits"], p["ids"], p["w"])
    bd.base_predict_cost(s["desc"], s["x"], B, p["ids"], p["w"], p["cost"])
    bd.base_select(s["desc"], B, p["ids"], p["cost"], case["budget"], p["scores"], p["counts"],
                   p["sel"], p["n_sel"], p["slot"])
    bd.base_moe_forward(s["desc"], s["x"], B, p["logits"], p["ids"], p["sel"], p["n_sel"],
                        p["slot"], case["budget"], case["flags"], s["residual"], s["y"], st["ws"])
    return dict(p, y=s["y"])


def work(case):
    d, I, E = case["d"], case["I"], case["E"]
    size = 4 if case.get("dtype") == "f32" else 2
    expert = 3 * d * I * size
    if case["kind"] == "pack":
        return {"bytes": 2 * E * expert, "flops": 0}
    B, K = case["B"], case["K"]
    if case["kind"] == "calib":
        pairs = case["batches"] * B * K
        return {"bytes": E * expert + E * d * d * 4 + 2 * E * d * 8 + case["batches"] * B * d * size
                + E * d * 4,
                "flops": 2 * pairs * 3 * d * I + pairs * d * d + 2 * case["batches"] * B * E * d}
    ns, kept = case["n_shared"], min(case["budget"], E, B * K)
    rows = E + (min(E, B * K) if case["rule"] == 0 else 0) + (1 if case["shared_gate"] else 0)
    moved = (kept + ns) * expert + rows * d * 4 + B * d * size * (3 if case["residual"] else 2)
    pairs = B * (min(K, kept) + ns)
    return {"bytes": case["layers"] * moved,
            "flops": case["layers"] * (2 * pairs * 3 * d * I + 2 * B * d * (E + K))}


def tolerance(case):
    if case["kind"] == "pack":
        return "exact"
    if case["kind"] == "calib":
        return {"rel": 8e-4}   # the targets carry the expert outputs' bf16 activations
    # fp32 layers: 32-bit sums.  bf16 layers: the activation and the output
    # are each rounded to bf16 once; ids and counts are whole and equal
    return {"rel": 1e-5} if case["dtype"] == "f32" else {"rel": 1e-2}


# ------------------------------------------------- the same in 64-bit torch --
def _ffn64(x, w13, w2):
    h = x @ w13.double().T
    I = w2.shape[1]
    return (torch.nn.functional.silu(h[:, :I]) * h[:, I:]) @ w2.double().T


def _route64(case, x, wr, br):
    l = x @ wr.double().T + br.double()
    top, ids = torch.sort(l, dim=1, descending=True, stable=True)
    K = case["K"]
    num = (l - top[:, :1]).exp()
    den = num.gather(1, ids[:, :K]).sum(1) if case.get("norm_topk", 1) else num.sum(1)
    return l, ids, num, den


def _layer64(case, seed, layer):
    E, K, B = case["E"], case["K"], case["B"]
    x = _tokens(case, seed, layer).double()
    l, order, num, den = _route64(case, x, *_router(case, seed, layer))
    ids = order[:, :K]
    w = num.gather(1, ids) / den[:, None]
    a, b = _predictor(case, seed, layer)
    rule = case["rule"]
    if rule == 1:
        cost = torch.zeros_like(w)
        cost[:, 0] = 1.0
    elif rule in (2, 3):
        cost = w ** (rule - 1)
    else:
        s = b.double()[ids]
        if rule == 0:
            n = x.norm(dim=1, keepdim=True).clamp_min(1e-300)
            s = s + ((x / n) @ a.double().T).gather(1, ids)
        cost = w * w * s.exp()
    scores = torch.zeros(E, dtype=torch.float64, device="cuda").index_add_(0, ids.flatten(),
                                                                         cost.flatten())
    routed = torch.zeros(E, dtype=torch.bool, device="cuda")
    routed[ids.flatten()] = True
    key = torch.where(routed, (scores > 0).double() if rule == 1 else scores, -1.0)
    n_sel = min(case["budget"], int(routed.sum()))
    kept = torch.zeros_like(routed)
    kept[torch.sort(key, descending=True, stable=True).indices[:n_sel]] = True
    # the executed experts: the K best kept ones, or the kept routes (drop)
    cand = kept[order]
    if case["flags"] & 2:
        cand[:, K:] = False
    take = cand & (cand.cumsum(1) <= K)
    execd = torch.zeros_like(take).scatter_(1, order, take)
    g = num * execd
    g = g / (g.sum(1, keepdim=True) if case["flags"] & 1 else den[:, None])
    g = torch.nan_to_num(g)
    y = _tokens(case, seed, layer, 7).double() if case["residual"] else torch.zeros_like(x)
    w13, w2 = _experts(case, seed, layer, E)
    for u in kept.nonzero().flatten().tolist():
        t = execd[:, u].nonzero().flatten()
        if len(t):
            y[t] += g[t, u, None] * _ffn64(x[t], w13[u], w2[u])
    sh = _shared(case, seed, layer)
    if sh is not None:
        gs = torch.sigmoid(x @ sh[2].double())[:, None] if sh[2] is not None else 1.0
        for i in range(case["n_shared"]):
            y += gs * _ffn64(x, sh[0][i], sh[1][i])
    return dict(logits=l, ids=None, w=w, cost=cost, scores=scores, counts=None, sel=None,
                n_sel=None, slot=None, y=y)


def exact(case, seed):
    if case["kind"] == "pack":
        E, d, I = case["E"], case["d"], case["I"]
        w13, w2 = _experts(case, seed, 0, E)
        # [gate/up][group][tile][row][k-step][quarter][8] to the fragment order
        a = w13.view(E, 2, I // 32, 2, 16, d // 32, 4, 8).permute(0, 2, 5, 1, 3, 6, 4, 7)
        b = w2.view(E, d // 64, 4, 16, I // 32, 4, 8).permute(0, 1, 4, 2, 5, 3, 6)
        return a.reshape(w13.shape).double(), b.reshape(w2.shape).double()
    if case["kind"] == "calib":
        E, d = case["E"], case["d"]
        wr, br = _router(case, seed, 0)
        w13, w2 = _experts(case, seed, 0, E)
        out = dict(head=torch.zeros(E, 4, dtype=torch.float64, device="cuda"),
                   sz=torch.zeros(E, d, dtype=torch.float64, device="cuda"),
                   q=torch.zeros(E, d, dtype=torch.float64, device="cuda"),
                   G=torch.zeros(E, d, d, dtype=torch.float64, device="cuda"))
        x = torch.cat([_tokens(case, seed, 0, 6 + b) for b in range(case["batches"])]).double()
        ids = _route64(case, x, wr, br)[1][:, :case["K"]]
        zb = x / x.norm(dim=1, keepdim=True)
        for u in range(E):
            t = (ids == u).any(1).nonzero().flatten()
            if not len(t):
                continue
            y = (_ffn64(x[t], w13[u], w2[u]).square().sum(1) + 1e-12).log()
            out["head"][u] = torch.stack([torch.full_like(y, 1).sum(), y.sum(), (y * y).sum(),
                                          torch.zeros_like(y[0])])
            out["sz"][u], out["q"][u] = zb[t].sum(0), y @ zb[t]
            out["G"][u] = zb[t].T @ zb[t]
        return out
    if case["staged"]:
        return _layer64(case, seed, 0)
    return [_layer64(case, seed, l)["y"] for l in range(case["layers"])]
