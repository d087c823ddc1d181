"""Performance cases of the framework: what a speculative-decoding program has
it do, through the Python entry points (`VerifyPass`, `DraftStep`, `expand`).

Three kinds of call:
  verify  one verify-MoE layer (`VerifyPass`): a batch of draft tokens is
          routed, gated, run through its experts and combined.  `fused` is
          the one-call form, otherwise the four calls; `packed` is the tile
          layout of the expert weights, otherwise row-major.
  draft   one draft step (`DraftStep`): every MoE layer of a model at k_draft
          experts per token, replayed from a HIP graph or enqueued eagerly.
  expand  routing-aware expansion of a batch of draft trees (`expand`).

Inputs are synthetic, drawn on the device from the seed: hidden states that
share a component across the batch, a router with unit-variance logits,
N(0, 0.02^2) expert weights (or uniform int4 codes of that spread), draft-tree
confidences, and draft trees of depth 8 and branch 4 whose tokens inherit
experts from their parents.  Verify and draft batches are redrawn until every
ranking decision is clear in 64 bits, so that two correct implementations
take the same decisions.
"""

import math

import torch

import paper_2608_15018_amd as s2
from paper_2608_15018_amd import draft as s2_draft

DEVICE = "cuda" if torch.cuda.is_available() else "cpu"

# Shapes: expert counts, k, cap and draft experts of the model table the
# workloads follow, sizes of the public architectures; "mixtral" and "tiny"
# are the repository's own layer workloads.
MODELS = {
    "mixtral": dict(hidden=4096, ffn=14336, n_experts=8, top_k=2, cap=4, rho=0.6),
    "qwen3": dict(hidden=2048, ffn=768, n_experts=128, top_k=8, cap=14, rho=0.5, layers=48,
                  k_draft=3),
    "deepseek": dict(hidden=2048, ffn=1408, n_experts=64, top_k=6, cap=16, n_shared=2,
                     ffn_shared=1408, rho=0.4, layers=26, k_draft=1),
    "olmoe": dict(hidden=2048, ffn=1024, n_experts=64, top_k=8, cap=18, rho=0.5, layers=16,
                  k_draft=2),
    "gptoss": dict(hidden=2880, ffn=2880, n_experts=128, top_k=4, cap=6, rho=0.5, layers=36,
                   k_draft=1),
    "tiny": dict(hidden=256, ffn=512, n_experts=8, top_k=2, cap=4, rho=0.0),
}
TREE_LAYERS = {"qwen3": (48, 128, 8), "deepseek": (26, 64, 6), "olmoe": (16, 64, 8),
               "gptoss": (36, 128, 4)}  # layers, experts, experts per token
DEPTH, BRANCH, BEAM = 8, 4, 4
T_AR, T_EXP, C_DRAFT = 512.0, 1.0, 16.0
DRAFT_WEIGHT_SETS = 4  # a draft step's layers cycle through this many weight sets
W_STD = 0.02


def _verify(model, wdt, B, alpha=0.5, packed=True, fused=True):
    return {"kind": "verify", "model": model, "wdt": wdt, "B": B, "alpha": alpha,
            "packed": packed, "fused": fused}


def _draft(model, wdt, B, graph):
    return {"kind": "draft", "model": model, "wdt": wdt, "B": B, "graph": graph}


def _expand(model, trees):
    return {"kind": "expand", "model": model, "trees": trees}


def listed():
    return [
        # The smallest verify call: a small fp32 layer, all launch latency.
        dict(_verify("tiny", "f32", 8, packed=False), name="tiny_f32_b8"),
        # One drafted token through a 48-layer model, as a serving loop replays it.
        dict(_draft("qwen3", "bf16", 1, True), name="draft_qwen3_bf16_b1"),
        # A draft-tree level of three tokens, quantised weights, enqueued eagerly.
        dict(_draft("olmoe", "q4g32", 3, False), name="draft_olmoe_q4_b3"),
        # One request's draft (length 8, width 2) against few, large experts.
        dict(_verify("mixtral", "bf16", 16), name="mixtral_bf16_b16"),
        # Two requests' drafts against many small experts.
        dict(_verify("qwen3", "bf16", 32), name="qwen3_bf16_b32"),
        # Four requests' drafts, routed and shared experts.
        dict(_verify("deepseek", "bf16", 64), name="deepseek_bf16_b64"),
        # A ragged batch on weights as a checkpoint stores them (row-major), the
        # four calls, sizes that are no power of two.
        dict(_verify("gptoss", "bf16", 37, packed=False, fused=False),
             name="gptoss_bf16_b37_rowmajor"),
        # The int4 layer at one request's draft and at four requests' drafts.
        dict(_verify("mixtral", "q4g32", 16), name="mixtral_q4_b16"),
        dict(_verify("mixtral", "q4g32", 64), name="mixtral_q4_b64"),
        # The largest batch: sixteen requests' drafts over every expert.
        dict(_verify("mixtral", "bf16", 256), name="mixtral_bf16_b256"),
        # Expansion of a single request's tree, and of a large serving batch.
        dict(_expand("olmoe", 1), name="expand_olmoe_t1"),
        dict(_expand("qwen3", 1024), name="expand_qwen3_t1024"),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    u = rng.random()
    if u < 0.2:
        return _expand(rng.choice(sorted(TREE_LAYERS)), _log_int(rng, 1, 1024))
    if u < 0.35:
        model = rng.choice(["qwen3", "deepseek", "olmoe", "gptoss"])
        wdt = "bf16" if model == "gptoss" else rng.choice(["bf16", "q4g32"])
        return _draft(model, wdt, rng.randint(1, 4), rng.random() < 0.5)
    if u < 0.42:
        return _verify("tiny", "f32", _log_int(rng, 1, 128), rng.choice([0.25, 0.5, 1.0]),
                       packed=False, fused=rng.random() < 0.5)
    model = rng.choice(["mixtral", "qwen3", "deepseek", "olmoe", "gptoss"])
    wdt = "bf16" if model == "gptoss" else rng.choice(["bf16", "q4g32"])
    packed = model == "mixtral" or rng.random() < 0.75
    most = 40 if model == "gptoss" else 256  # beyond, it streams more than any listed case
    return _verify(model, wdt, _log_int(rng, 1, most), rng.choice([0.0, 0.5, 1.0]), packed,
                   rng.random() < 0.75)


# ------------------------------------------------------------------- inputs


def _gen(*key):
    g = torch.Generator(device=DEVICE)
    s = 0
    for k in key:
        s = (s * 1_000_003 + int(k) + 1) & 0x7FFFFFFFFFFFFFFF
    g.manual_seed(s)
    return g


def _matrices(n, rows, cols, wdt, g):
    """n expert matrices [rows, cols] (and int4 scales)."""
    if wdt == "q4g32":
        codes = torch.randint(0, 256, (n, rows, cols // 2), generator=g, device=DEVICE,
                              dtype=torch.uint8)
        scales = torch.rand((n, rows, cols // 32), generator=g, device=DEVICE)
        return codes, scales.mul_(0.5).add_(0.75).mul_(W_STD / 4.61).to(torch.float16)
    dt = torch.bfloat16 if wdt == "bf16" else torch.float32
    return torch.randn((n, rows, cols), generator=g, device=DEVICE, dtype=dt).mul_(W_STD), None


def _experts(n, F, H, wdt, *key):
    """Weights of n experts, row-major: gate, up [n, F, H], down [n, H, F]."""
    out = {}
    for t, (name, rows, cols) in enumerate((("gate", F, H), ("up", F, H), ("down", H, F))):
        out[name], scales = _matrices(n, rows, cols, wdt, _gen(*key, t))
        if scales is not None:
            out[name + "_s"] = scales
    return out


def _weights(m, wdt, *key):
    """(routed, shared) weight dicts of one layer of model m."""
    routed = _experts(m["n_experts"], m["ffn"], m["hidden"], wdt, *key, 1)
    S = m.get("n_shared", 0)
    return routed, (_experts(S, m["ffn_shared"], m["hidden"], wdt, *key, 2) if S else {})


def _confidences(B, g):
    """w_b of ceil(B / 8) chains: running products of Beta(5, 1) edges."""
    D = min(8, B)
    q = torch.rand((-(-B // D), D), generator=g, device=DEVICE) ** (1.0 / 5.0)
    return torch.cumprod(q, 1).reshape(-1)[:B].contiguous()


def _clear(r, k, cap, E):
    """Whether every ranking of the batch is decided by a margin that 32-bit
    arithmetic cannot cross."""
    def margin(v, n):
        s = v.sort(dim=-1, descending=True).values
        return float((s[..., n - 1] - s[..., n]).min())
    ok = margin(r["logits"], k) > 1e-5 and margin(r["logits"], k + 1 if k + 1 < E else k) > 1e-5
    ok = ok and margin(r["biased"], k) > 1e-5
    return ok and (cap >= E or margin(r["g"], cap) > 1e-4)


def _route64(x, router, conf, k, cap, alpha):
    """The routing of one batch in 64 bits."""
    E = router.shape[0]
    ell = x.double() @ router.double().T
    w = conf.double().clamp(min=0)
    top = ell.topk(k + 1, dim=-1).values
    gap = top[:, 0] - top[:, k]
    g = w @ ell
    pref = torch.zeros(E, dtype=torch.bool, device=ell.device)
    if bool((w > 0).any()):
        pref[g.topk(cap).indices] = True
    biased = ell + alpha * gap[:, None] * pref
    idx = biased.topk(k, dim=-1).indices.sort(dim=-1).values
    return {"logits": ell, "gap": gap, "g": g, "biased": biased, "idx": idx,
            "gate_w": torch.softmax(ell.gather(1, idx), dim=-1)}


def _batch(m, act, B, k, cap, alpha, *key):
    """x, router, confidences and their 64-bit routing; redrawn until clear."""
    H, E = m["hidden"], m["n_experts"]
    dt = torch.float32 if act == "f32" else torch.bfloat16
    for attempt in range(50):
        g = _gen(*key, 100, attempt)
        u = torch.randn(H, generator=g, device=DEVICE)
        n = torch.randn((B, H), generator=g, device=DEVICE)
        x = (m["rho"] ** 0.5 * u + (1 - m["rho"]) ** 0.5 * n).to(dt)
        router = (torch.randn((E, H), generator=g, device=DEVICE) / H ** 0.5).to(dt)
        conf = _confidences(B, g)
        r = _route64(x, router, conf, k, cap, alpha)
        if _clear(r, k, cap, E):
            return x, router, conf, r
    raise RuntimeError("no batch with clear rankings")


def _verify_batch(case, seed):
    m = MODELS[case["model"]]
    act = "f32" if case["wdt"] == "f32" else "bf16"
    return _batch(m, act, case["B"], m["top_k"], m["cap"], case["alpha"], seed, 7)


def _draft_batch(case, seed, layer):
    m = MODELS[case["model"]]
    return _batch(m, "bf16", case["B"], m["k_draft"], m["k_draft"], 0.0, seed, 8, layer)


def _gamma(alpha, shape, g):
    return torch._standard_gamma(torch.full(shape, alpha, device=DEVICE), generator=g)


def _trees(case, seed):
    """A padded batch of draft trees.  Each level's first 2 to 4 nodes (a
    number of the tree's own) are expanded into 4 children; a child keeps
    each of its parent's experts with probability 0.6 and draws the rest from
    a Zipf popularity of its tree and layer."""
    T = case["trees"]
    L, E, k = TREE_LAYERS[case["model"]]
    g = _gen(seed, 9)
    N = BRANCH + (DEPTH - 1) * BEAM * BRANCH
    beam = torch.randint(2, BEAM + 1, (T,), generator=g, device=DEVICE)
    zipf = -1.1 * torch.log(torch.arange(1, E + 1, device=DEVICE, dtype=torch.float32))
    order = torch.rand((T, L, E), generator=g, device=DEVICE).argsort(dim=-1)
    logp = torch.empty((T, L, E), device=DEVICE).scatter_(2, order, zipf.expand(T, L, E))

    def draw_ids(n, keep):
        """k distinct experts per tree, node and layer (Gumbel top-k), those in keep first."""
        key = torch.rand((T, n, L, E), generator=g, device=DEVICE).clamp_(1e-9, 1 - 1e-7)
        key = key.log_().neg_().log_().neg_().add_(logp[:, None])
        if keep is not None:
            key.masked_fill_(keep, float("inf"))
        return key.topk(k, dim=-1).indices

    root = draw_ids(1, None)[:, 0]
    parent = torch.full((T, N), -1, dtype=torch.int32, device=DEVICE)
    q = torch.zeros((T, N), device=DEVICE)
    eid = torch.full((T, N, L, k), -1, dtype=torch.int32, device=DEVICE)
    tree = torch.arange(T, device=DEVICE)
    prev = root[:, None]  # expert ids of the nodes that this level expands
    for level in range(DEPTH):
        S = 1 if level == 0 else BEAM
        up = prev.repeat_interleave(BRANCH, dim=1)
        kept = torch.rand(up.shape, generator=g, device=DEVICE) < 0.6
        keep = torch.zeros((T, S * BRANCH, L, E), dtype=torch.bool, device=DEVICE)
        keep.scatter_(3, up, kept)
        ids = draw_ids(S * BRANCH, keep)
        a, b = _gamma(4.0, (T, S), g), _gamma(1.2, (T, S), g)
        first = (a / (a + b)).clamp(0, 1)
        rest = _gamma(0.3, (T, S, 31), g)
        rest = (rest / rest.sum(-1, keepdim=True)).sort(dim=-1, descending=True).values
        conf = torch.cat([first[..., None], rest[..., :BRANCH - 1] * (1 - first[..., None])], -1)
        for s in range(S):
            base = 0 if level == 0 else BRANCH + (level - 1) * BRANCH * beam + s * BRANCH
            if level == 0:
                above = torch.full((T,), -1, device=DEVICE)
            else:
                above = (0 if level == 1 else BRANCH + (level - 2) * BRANCH * beam) + s + 0 * beam
            live = (s < beam) if level else torch.ones_like(beam, dtype=torch.bool)
            for c in range(BRANCH):
                at = (base + c + 0 * beam)[live]
                t = tree[live]
                parent[t, at] = above[live].to(torch.int32)
                q[t, at] = conf[live, s, c]
                eid[t, at] = ids[live, s * BRANCH + c].to(torch.int32)
        prev = ids[:, :BEAM]
    return {"parent": parent, "q": q, "eid": eid, "root_eid": root.to(torch.int32).contiguous(),
            "c_draft": torch.full((T, N), C_DRAFT, device=DEVICE),
            "n_nodes": (BRANCH + (DEPTH - 1) * BRANCH * beam).to(torch.int32)}


# ------------------------------------------------------------ prepare and run


def _layer_of(m, wdt, k, cap, alpha, packed):
    return s2.make_layer(hidden=m["hidden"], ffn=m["ffn"], n_experts=m["n_experts"], top_k=k,
                         n_shared=m.get("n_shared", 0), ffn_shared=m.get("ffn_shared", 0),
                         cap=cap, alpha=alpha, act="f32" if wdt == "f32" else "bf16", wdt=wdt,
                         flags=s2.PACKED_WEIGHTS if packed else 0)


def prepare(case, seed):
    if case["kind"] == "expand":
        d = _trees(case, seed)
        T, N = d["parent"].shape
        return {"kind": "expand", "in": d, "out": s2.ExpandOut(T, N),
                "E": TREE_LAYERS[case["model"]][1]}
    m, wdt = MODELS[case["model"]], case["wdt"]
    if case["kind"] == "verify":
        layer = _layer_of(m, wdt, m["top_k"], m["cap"], case["alpha"], case["packed"])
        dev = _weights(m, wdt, seed, 0)
        if case["packed"]:
            dev, w = s2.pack_expert_weights(dev, wdt)
        else:
            w = s2.make_weights(*dev)
        x, router, conf, _ = _verify_batch(case, seed)
        return {"kind": "verify", "pass": s2.VerifyPass(layer, case["B"], fused=case["fused"]),
                "args": (x, router, conf, w), "keep": dev}
    layer = s2_draft.draft_layer(case["model"], wdt)
    sets = []
    for j in range(min(DRAFT_WEIGHT_SETS, m["layers"])):
        sets.append(s2.pack_expert_weights(_weights(m, wdt, seed, j), wdt))
    inputs = []
    for l in range(m["layers"]):
        x, router, _, _ = _draft_batch(case, seed, l)
        inputs.append((x, router, sets[l % len(sets)][1]))
    step = s2_draft.DraftStep(layer, case["B"], inputs)
    if case["graph"]:
        step.capture()
    return {"kind": "draft", "step": step, "graph": case["graph"], "keep": sets}


ROUTING = ("logits", "gap", "plain_idx", "g", "pref", "idx", "gate_w", "count", "offset", "slot",
           "uniq", "n_uniq")


def run(state):
    if state["kind"] == "expand":
        d, out = state["in"], state["out"]
        s2.expand(d["parent"], d["q"], d["eid"], d["c_draft"], d["n_nodes"], out, state["E"],
                  T_AR, T_EXP, root_eid=d["root_eid"])
        return {n: getattr(out, n) for n in ("order", "util", "n_new", "n_admit", "n_pairs",
                                             "status")}
    if state["kind"] == "draft":
        step = state["step"]
        if state["graph"]:
            step.replay()
        else:
            step()
        return step.outputs()
    p = state["pass"]
    y = p(*state["args"])
    return {"y": y, "expert_out": p.expert_out, **{n: getattr(p.rt, n) for n in ROUTING}}


# ------------------------------------------------------ work, tolerance, exact


def _matrix_bytes(n, wdt):
    return n * {"f32": 4, "bf16": 2, "q4g32": 0.5 + 2 / 32}[wdt]


def _layer_work(m, wdt, B, k, n_active):
    """Each activated expert's weights, the router, x and the confidences read
    once; the routing arrays, expert_out and y written once."""
    H, F, E = m["hidden"], m["ffn"], m["n_experts"]
    S, Fs = m.get("n_shared", 0), m.get("ffn_shared", 0)
    act = 4 if wdt == "f32" else 2
    weights = _matrix_bytes(3 * H * (n_active * F + S * Fs), wdt)
    io = act * H * (E + B) + 4 * B + 4 * B * H * (k + S + 1) + 4 * (B * (E + 1 + 4 * k) + 6 * E)
    flops = 2 * B * H * E + 6 * B * H * (k * F + S * Fs)
    return weights + io, flops


def _n_active(batches):
    """Mean number of experts that the given 64-bit routings activate."""
    n = [int(torch.unique(b[3]["idx"]).numel()) for b in batches]
    return sum(n) / len(n)


def work(case):
    """Bytes and operations of one pass.  The experts a batch activates vary
    with its draw (4 to 8 of 8 at the Mixtral shape), so their number is a mean
    over several."""
    if case["kind"] == "expand":
        L, E, k = TREE_LAYERS[case["model"]]
        T, N = case["trees"], BRANCH + (DEPTH - 1) * BEAM * BRANCH
        nodes = T * (BRANCH + (DEPTH - 1) * BRANCH * 3)  # 2 to 4 expanded nodes a level
        return {"bytes": nodes * (12 + 4 * L * k) + T * (4 * L * k + 4 + N * 16 + 12), "flops": 0}
    m, wdt, B = MODELS[case["model"]], case["wdt"], case["B"]
    if case["kind"] == "verify":
        n = _n_active([_verify_batch(case, seed) for seed in range(24)])
        b, f = _layer_work(m, wdt, B, m["top_k"], n)
        return {"bytes": b, "flops": f}
    n = _n_active([_draft_batch(case, 1, l) for l in range(m["layers"])])
    b, f = _layer_work(m, wdt, B, m["k_draft"], n)
    return {"bytes": b * m["layers"], "flops": f * m["layers"]}


def tolerance(case):
    """Expansion: integers, and 64-bit utilities whose operations and order the
    interface fixes.  Layers: about four times the distance from the 64-bit
    result, which the rounding of the SwiGLU activations sets (bf16, or fp16
    with int4 weights)."""
    if case["kind"] == "expand":
        return "exact"
    return {"rel": {"f32": 2e-6, "bf16": 8e-3, "q4g32": 2e-3}[case["wdt"]]}


def _dense64(routed, name, e):
    """Matrix of expert e in 64 bits."""
    w = routed[name][e]
    if name + "_s" not in routed:
        return w.double()
    c = torch.stack([w & 15, w >> 4], dim=-1).reshape(w.shape[0], -1).double() - 8.0
    return c * routed[name + "_s"][e].double().repeat_interleave(32, dim=1)


def _ffn64(weights, e, x):
    h = x @ _dense64(weights, "gate", e).T
    h = h * torch.sigmoid(h) * (x @ _dense64(weights, "up", e).T)
    return h @ _dense64(weights, "down", e).T


def _layer64(m, weights, x, r, k):
    """(expert_out, y) of one layer in 64 bits."""
    routed, shared = weights
    B, S, x = x.shape[0], m.get("n_shared", 0), x.double()
    out = torch.zeros((B * k + S * B, m["hidden"]), dtype=torch.float64, device=x.device)
    for e in torch.unique(r["idx"]).tolist():
        b, j = (r["idx"] == e).nonzero(as_tuple=True)
        out[b * k + j] = _ffn64(routed, e, x[b])
    for s in range(S):
        out[B * k + s * B:B * k + (s + 1) * B] = _ffn64(shared, s, x)
    y = (out[:B * k].reshape(B, k, -1) * r["gate_w"][..., None]).sum(1)
    return out, y + out[B * k:].reshape(S, B, m["hidden"]).sum(0)


def _expand64(case, seed):
    d = _trees(case, seed)
    L, E, _ = TREE_LAYERS[case["model"]]
    T, N = d["parent"].shape
    dev = d["parent"].device
    res = {"order": torch.full((T, N), -1, dtype=torch.int32, device=dev),
           "util": torch.zeros((T, N), dtype=torch.float64, device=dev),
           "n_new": torch.zeros((T, N), dtype=torch.int32, device=dev),
           "n_admit": torch.zeros(T, dtype=torch.int32, device=dev),
           "n_pairs": torch.zeros(T, dtype=torch.int32, device=dev),
           "status": torch.zeros(T, dtype=torch.int32, device=dev)}
    node = torch.arange(N, device=dev)
    for t0 in range(0, T, 64):
        sl = slice(t0, min(T, t0 + 64))
        par, eid = d["parent"][sl].long(), d["eid"][sl].long()
        n = par.shape[0]
        rows = torch.zeros((n, N, L, E + 1), dtype=torch.bool, device=dev)
        rows.scatter_(3, torch.where(eid < 0, E, eid), True)
        rows = rows[..., :E]
        union = torch.zeros((n, L, E), dtype=torch.bool, device=dev)
        union.scatter_(2, d["root_eid"][sl].long(), True)
        p = torch.ones((n, N), dtype=torch.float64, device=dev)
        for i in range(N):
            above = p.gather(1, par[:, i:i + 1].clamp(min=0))[:, 0]
            p[:, i] = torch.where(par[:, i] < 0, torch.ones_like(above), above) * d["q"][sl, i].double()
        benefit, cost = p * T_AR, d["c_draft"][sl].double()
        real = node[None] < d["n_nodes"][sl, None]
        admitted = torch.zeros((n, N), dtype=torch.bool, device=dev)
        going = torch.ones(n, dtype=torch.bool, device=dev)
        for step in range(N):
            new = (rows & ~union[:, None]).sum((2, 3))
            util = benefit / (new.double() * T_EXP + cost)
            open_ = real & ~admitted & ((par < 0) | admitted.gather(1, par.clamp(min=0)))
            util = torch.where(open_, util, torch.full_like(util, -1.0))
            best = util.max(1).values
            j = torch.where(util == best[:, None], node[None], N).min(1).values
            going = going & (best >= 1.0)
            if not bool(going.any()):
                break
            t = going.nonzero()[:, 0]
            res["order"][sl][t, step] = j[t].to(torch.int32)
            res["util"][sl][t, step] = best[t]
            res["n_new"][sl][t, step] = new[t, j[t]].to(torch.int32)
            res["n_admit"][sl][t] += 1
            admitted[t, j[t]] = True
            union[t] |= rows[t, j[t]]
        res["n_pairs"][sl] = union.sum((1, 2)).to(torch.int32)
    return res


def exact(case, seed):
    if case["kind"] == "expand":
        return _expand64(case, seed)
    m, wdt = MODELS[case["model"]], case["wdt"]
    if case["kind"] == "verify":
        x, _, _, r = _verify_batch(case, seed)
        out, y = _layer64(m, _weights(m, wdt, seed, 0), x, r, m["top_k"])
        known = {n: r[n] for n in ("logits", "gap", "g", "gate_w")}
        return {"y": y, "expert_out": out, **{n: known.get(n) for n in ROUTING}}
    ys = [None] * m["layers"]
    for j in range(min(DRAFT_WEIGHT_SETS, m["layers"])):
        weights = _weights(m, wdt, seed, j)
        for l in range(j, m["layers"], DRAFT_WEIGHT_SETS):
            x, _, _, r = _draft_batch(case, seed, l)
            ys[l] = _layer64(m, weights, x, r, m["k_draft"])[1]
    return ys
