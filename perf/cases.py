"""The work that a serving program has libmoe do, as measurable cases.

A case is a dict of plain values; `kind` names the call a program makes:

  layer     MoeLayer.forward: routing, permutation, expert FFN and combine of
            one GPU's share of an MoE layer (a TP slice of every expert, or an
            EP slice of whole experts), with every buffer kept by the layer;
  ffn       grouped_ffn on rows that already lie expert by expert, as an EP
            rank gets them from the dispatch all-to-all;
  dispatch  route, then permute with the row gather: what an EP rank does
            with its own tokens before that all-to-all;
  combine   combine of the rows that came back, with a shared expert's rows;
  reshard   reshard_experts: one layer's expert weights from the EP to the TP
            view or back, in a layout switch;
  kv        kv_slots for both sides of a layout switch, then kv_move for each
            layer.

Shapes are those of the repository's workloads (Mixtral-, Qwen-MoE-, Qwen3-
and DeepSeek-V3-shaped layers and the tiny replicated one), of their slices
over 2 to 8 ranks, and generic layers whose sizes are only multiples of 8.
Inputs follow moe_inputs: x ~ N(0, 1), logits of unit deviation (with a Zipf
popularity where a layer is skewed), weights ~ N(0, 0.02^2), drawn on the GPU.
"""
import math

import numpy as np
import torch

import paper_2606_26607_amd as moe

DEV = "cuda:0"

# H, E, k, I, shared expert
MODELS = {
    "tiny": (256, 8, 2, 512, False),
    "mixtral": (4096, 8, 2, 14336, False),
    "qwen-moe": (2048, 128, 8, 768, False),
    "qwen3": (4096, 128, 8, 1536, False),
    "dsv3": (7168, 256, 8, 2048, True),
}


def _layer(model, T, layout, P, rank=0, zipf=0.0, shared=None):
    H, E, k, I, has_shared = MODELS[model]
    return {"kind": "layer", "T": T, "H": H, "E": E, "k": k, "I": I, "layout": layout, "P": P, "rank": rank,
            "zipf": zipf, "shared": (has_shared and layout == "ep") if shared is None else shared}


def listed():
    return [
        # the smallest call: a 64-token batch of a small replicated layer, bound by launches and latency
        {"name": "tiny-64", **_layer("tiny", 64, "replicated", 1)},
        # prefill on a TP = 8 rank: every expert's slice, all tokens
        {"name": "mixtral-tp8-4096", **_layer("mixtral", 4096, "tp", 8)},
        # prefill on an EP = 8 rank with one large expert
        {"name": "mixtral-ep8-4096", **_layer("mixtral", 4096, "ep", 8)},
        # prefill on an EP = 8 rank with 16 small experts under a skewed load
        {"name": "qwen-moe-ep8-8192", **_layer("qwen-moe", 8192, "ep", 8, zipf=1.2)},
        # the same layer in the other view: 128 slices of width 96, a ragged chunk of tokens
        {"name": "qwen-moe-tp8-2051", **_layer("qwen-moe", 2051, "tp", 8, rank=3)},
        # decode on an EP = 8 rank: 32 experts and the shared one, bound by the weights
        {"name": "dsv3-ep8-64", **_layer("dsv3", 64, "ep", 8)},
        # decode on a TP = 8 rank: 128 slices of width 192
        {"name": "qwen3-tp8-128", **_layer("qwen3", 128, "tp", 8)},
        # the expert FFN alone on received rows: 16 experts, a ragged number of rows, uneven loads
        {"name": "ffn-qwen3-ep8-3001", "kind": "ffn", "n": 3001, "El": 16, "H": 4096, "I": 1536, "skew": 0.7},
        # a rank's own tokens sorted for the all-to-all
        {"name": "dispatch-dsv3-2048", "kind": "dispatch", "T": 2048, "H": 7168, "E": 256, "k": 8},
        # the rows that come back, added up with the shared expert's
        {"name": "combine-dsv3-2048", "kind": "combine", "T": 2048, "H": 7168, "E": 256, "k": 8, "shared": True},
        # a layout switch: one layer's weights into rank 5's TP view, from all 8 ranks' EP views
        {"name": "reshard-qwen3-ep-tp", "kind": "reshard", "dir": "ep_to_tp", "E": 128, "H": 4096, "I": 1536, "P": 8,
         "rank": 5, "own": False},
        # ... and two layers' KV pages of 256 requests into a TP rank's pool
        {"name": "kv-256req-ep-tp", "kind": "kv", "dir": "ep_to_tp", "requests": 256, "lo": 500, "hi": 3500,
         "heads": 4, "head_dim": 128, "page": 16, "P": 8, "layers": 2},
    ]


# no drawn case moves or computes more than the largest listed ones
MOST_FLOPS, MOST_BYTES, MOST_WEIGHTS = 3.6e11, 2.6e9, 3.0e9


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw(rng):
    kind = rng.choices(["layer", "ffn", "dispatch", "combine", "reshard", "kv"], [10, 3, 2, 2, 1, 1])[0]
    model = rng.choice(["mixtral", "qwen-moe", "qwen3", "dsv3", "generic"])
    if model == "generic":  # any multiples of 8
        H, E, k, shared = 8 * _log(rng, 16, 640), 8 * rng.randint(1, 12), rng.randint(1, 8), False
    else:
        H, E, k, I, shared = MODELS[model]
    P = rng.choice([2, 4, 8])
    if model == "generic":
        I = 8 * P * _log(rng, 4, 256)
    T = _log(rng, 1, 8192)
    if kind == "layer":
        layout = rng.choice(["tp", "ep"])
        return {"kind": "layer", "T": T, "H": H, "E": E, "k": k, "I": I, "layout": layout, "P": P,
                "rank": rng.randrange(P), "zipf": rng.choice([0.0, 0.0, 1.2]),
                "shared": shared and layout == "ep" and T >= P}
    if kind == "ffn":
        return {"kind": "ffn", "n": _log(rng, 8, 16384), "El": E // P, "H": H, "I": I,
                "skew": rng.choice([0.0, 0.7, 1.2])}
    if kind == "dispatch":
        return {"kind": "dispatch", "T": T, "H": H, "E": E, "k": k}
    if kind == "combine":
        return {"kind": "combine", "T": T, "H": H, "E": E, "k": k, "shared": shared}
    if kind == "reshard":
        return {"kind": "reshard", "dir": rng.choice(["ep_to_tp", "tp_to_ep"]), "E": E, "H": H, "I": I, "P": P,
                "rank": rng.randrange(P), "own": rng.choice([False, True])}
    hi = _log(rng, 64, 4096)
    return {"kind": "kv", "dir": rng.choice(["ep_to_tp", "tp_to_ep"]), "requests": _log(rng, 8, 256),
            "lo": max(1, hi // 7), "hi": hi, "heads": rng.choice([4, 8]), "head_dim": rng.choice([64, 128]),
            "page": rng.choice([16, 64]), "P": P, "layers": rng.randint(1, 4)}


def draw(rng):
    while True:
        c = _draw(rng)
        w = work(c)
        weights = 0
        if c["kind"] in ("layer", "ffn", "reshard"):
            El, Is = _slice(c) if c["kind"] == "layer" else (c.get("El") or c["E"] // c["P"], c["I"])
            weights = 6 * El * c["H"] * Is
        if w["flops"] <= MOST_FLOPS and w["bytes"] <= MOST_BYTES and weights <= MOST_WEIGHTS:
            return c


# ------------------------------------------------------------------ sizes
def _slice(c):
    """(local experts, expert width) of a layer case's rank."""
    if c["layout"] == "ep":
        return c["E"] // c["P"], c["I"]
    return c["E"], c["I"] // c["P"]


def _bias(c):
    """Log popularity of the experts: a property of the layer, the same for every batch."""
    b = np.zeros(c["E"], np.float32)
    if c["zipf"]:
        rank = np.random.default_rng(1003).permutation(c["E"]) + 1
        b = (-c["zipf"] * np.log(rank)).astype(np.float32)
    return b


def _share(c):
    """(pairs on this rank, experts with rows), from a sample of at most 1024 tokens."""
    El, _ = _slice(c)
    n = min(c["T"], 1024)
    lg = np.random.default_rng(7).standard_normal((n, c["E"]), np.float32) + _bias(c)
    ids = np.argpartition(-lg, c["k"] - 1, axis=1)[:, :c["k"]]
    e0 = c["rank"] * El if c["layout"] == "ep" else 0
    cnt = np.bincount(ids.ravel(), minlength=c["E"])[e0:e0 + El]
    return max(1, int(cnt.sum() * c["T"] / n)), max(1, int(np.sum(cnt > 0)))


def _rows(c):
    """Rows of each expert of an ffn case: uneven with a Zipf exponent `skew`, a property of the layer."""
    p = (np.random.default_rng(11).permutation(c["El"]) + 1.0) ** -c["skew"]
    return p / p.sum()


def _lengths(c):
    rng = np.random.default_rng(2606)
    return rng.integers(c["lo"], c["hi"] + 1, c["requests"]), rng.integers(0, c["P"], c["requests"])


def _kv_heads(c):
    """KV heads that one TP rank holds."""
    return max(1, c["heads"] // c["P"])


def work(case):
    c = case
    if c["kind"] == "layer":
        El, Is = _slice(c)
        n, active = _share(c)
        T, H = c["T"], c["H"]
        sc = T // c["P"] if c["shared"] else 0
        b = 2 * T * H * 2 + T * c["E"] * 4 + T * c["k"] * 8 + (active + (1 if sc else 0)) * 6 * H * Is
        return {"bytes": b, "flops": 6 * H * Is * (n + sc)}
    if c["kind"] == "ffn":
        active = float(np.sum(1 - (1 - _rows(c)) ** c["n"]))
        return {"bytes": 4 * c["n"] * c["H"] + active * 6 * c["H"] * c["I"] + 4 * (c["El"] + 1),
                "flops": 6 * c["n"] * c["H"] * c["I"]}
    if c["kind"] == "dispatch":
        T, k = c["T"], c["k"]
        return {"bytes": T * c["E"] * 4 + 2 * T * c["H"] * (1 + k) + T * k * 16 + 8 * c["E"], "flops": 0}
    if c["kind"] == "combine":
        T, k = c["T"], c["k"]
        return {"bytes": 2 * T * c["H"] * (1 + k + (1 if c["shared"] else 0)) + T * k * 8,
                "flops": 2 * T * c["H"] * k}
    if c["kind"] == "reshard":
        n = 3 * c["E"] * c["H"] * (c["I"] // c["P"]) // (c["P"] if c["own"] else 1)
        return {"bytes": 4 * n, "flops": 0}
    lengths, owner = _lengths(c)
    tok = int(lengths.sum() if c["dir"] == "ep_to_tp" else lengths[owner == owner[0]].sum())
    heads = _kv_heads(c) if c["dir"] == "ep_to_tp" else c["heads"]
    return {"bytes": c["layers"] * tok * heads * c["head_dim"] * 2 * 2 * 2 + tok * 16, "flops": 0}


# ----------------------------------------------------------------- inputs
def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _normal(g, shape, std=1.0):
    t = torch.randn(shape, generator=g, device=DEV, dtype=torch.bfloat16)
    return t if std == 1.0 else t.mul_(std)


def _layer_inputs(c, seed):
    """x, logits, w13, w2 (and the shared expert's pair)."""
    g = _gen(seed)
    El, Is = _slice(c)
    x = _normal(g, (c["T"], c["H"]))
    logits = torch.randn((c["T"], c["E"]), generator=g, device=DEV) + torch.from_numpy(_bias(c)).to(DEV)
    w13, w2 = _normal(g, (El, 2 * Is, c["H"]), 0.02), _normal(g, (El, c["H"], Is), 0.02)
    sw13 = sw2 = None
    if c["shared"]:
        sw13, sw2 = _normal(g, (1, 2 * Is, c["H"]), 0.02), _normal(g, (1, c["H"], Is), 0.02)
    return x, logits, w13, w2, sw13, sw2


def _shared_rows(c):
    """The token rows that the rank's shared expert takes: its data-parallel share."""
    n = c["T"] // c["P"] if c["shared"] else 0
    return c["rank"] * n, n


def _ffn_inputs(c, seed):
    g = _gen(seed)
    counts = np.random.default_rng(seed).multinomial(c["n"], _rows(c))
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    x = _normal(g, (c["n"], c["H"]))
    return x, offsets, _normal(g, (c["El"], 2 * c["I"], c["H"]), 0.02), _normal(g, (c["El"], c["H"], c["I"]), 0.02)


def _dispatch_inputs(c, seed):
    g = _gen(seed)
    return _normal(g, (c["T"], c["H"])), torch.randn((c["T"], c["E"]), generator=g, device=DEV)


def _combine_inputs(c, seed):
    g = _gen(seed)
    T, k, H = c["T"], c["k"], c["H"]
    y = _normal(g, (T * k, H))
    p, ids = torch.softmax(torch.randn((T, c["E"]), generator=g, device=DEV), 1).topk(k, 1)
    w = (p / p.sum(1, keepdim=True)).contiguous()
    order = torch.sort(ids.reshape(-1), stable=True).indices  # rows lie expert by expert
    p2r = torch.empty(T * k, dtype=torch.int32, device=DEV)
    p2r[order] = torch.arange(T * k, dtype=torch.int32, device=DEV)
    sy = _normal(g, (T, H)) if c["shared"] else None
    return y, p2r, w, sy


def _tables(rng, lengths, page, width):
    """Page tables of a pool's requests, its pages shuffled; and the pool's pages."""
    need = -(-lengths // page)
    pages = int(need.sum()) + 8
    perm = rng.permutation(pages).astype(np.int32)
    tab = np.zeros((len(lengths), width), np.int32)
    at = 0
    for i, m in enumerate(need):
        tab[i, :m] = perm[at:at + m]
        at += m
    return tab, pages


def _up(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def _kv_state(c, seed):
    """ep_to_tp: the EP pools of all ranks into rank 0's TP pool.  tp_to_ep: the TP pools of all heads into one
    rank's EP pool, for the requests it takes over."""
    g, rng = _gen(seed), np.random.default_rng(seed)
    lengths, owner = _lengths(c)
    D, L, page, P = c["head_dim"], c["layers"], c["page"], c["P"]
    width = int(-(-lengths.max() // page))
    pool = lambda pages, heads: [_normal(g, (pages * page, heads, D)) for _ in range(L)]  # noqa: E731
    zero = lambda pages, heads: [torch.zeros((pages * page, heads, D), dtype=torch.bfloat16, device=DEV)  # noqa: E731
                                 for _ in range(L)]
    nh = _kv_heads(c)
    if c["dir"] == "ep_to_tp":
        ranks = [q for q in range(P) if (owner == q).any()]
        ls = np.concatenate([lengths[owner == q] for q in ranks])
        tabs = [_tables(rng, lengths[owner == q], page, width) for q in ranks]
        src_tab = np.concatenate([t for t, _ in tabs])
        src = [(pool(n, c["heads"]), pool(n, c["heads"])) for _, n in tabs]
        counts = [int(lengths[owner == q].sum()) for q in ranks]
        dst_tab, n = _tables(rng, ls, page, width)
        dst = (zero(n, nh), zero(n, nh))
    else:
        ls = lengths[owner == owner[0]]
        src_tab, n = _tables(rng, ls, page, width)
        src = [(pool(n, nh), pool(n, nh)) for _ in range(c["heads"] // nh)]
        counts = [int(ls.sum())] * len(src)
        dst_tab, n = _tables(rng, ls, page, width)
        dst = (zero(n, c["heads"]), zero(n, c["heads"]))
    tok = int(ls.sum())
    return {"src": src, "dst": dst, "counts": counts, "src_tab": _up(src_tab), "dst_tab": _up(dst_tab),
            "first": _up(np.concatenate([[0], np.cumsum(ls)]).astype(np.int32)), "heads": nh,
            "slot_src": torch.empty(tok, dtype=torch.int32, device=DEV),
            "slot_dst": torch.empty(tok, dtype=torch.int32, device=DEV)}


def prepare(case, seed):
    c = case
    if c["kind"] == "layer":
        x, logits, w13, w2, sw13, sw2 = _layer_inputs(c, seed)
        sb, sc = _shared_rows(c)
        e0 = c["rank"] * w13.shape[0] if c["layout"] == "ep" else 0
        layer = moe.MoeLayer(c["T"], c["E"], c["k"], e0, w13, w2, sw13, sw2, sb, sc)
        return {"case": c, "layer": layer, "x": x, "logits": logits}
    if c["kind"] == "ffn":
        x, offsets, w13, w2 = _ffn_inputs(c, seed)
        ws = torch.empty(moe.ffn_workspace_size(c["n"], c["El"], c["H"], c["I"]), dtype=torch.uint8, device=DEV)
        return {"case": c, "x": x, "offsets": _up(offsets), "w13": w13, "w2": w2, "ws": ws, "y": torch.empty_like(x)}
    if c["kind"] == "dispatch":
        x, logits = _dispatch_inputs(c, seed)
        T, E, k = c["T"], c["E"], c["k"]
        i32 = lambda *s: torch.zeros(s, dtype=torch.int32, device=DEV)  # noqa: E731
        bufs = {"counts": i32(E), "offsets": i32(E + 1), "row_to_pair": i32(T * k), "pair_to_row": i32(T * k),
                "x_perm": torch.empty((T * k, c["H"]), dtype=torch.bfloat16, device=DEV)}
        ws = torch.empty(moe.permute_workspace_size(T, k, E), dtype=torch.uint8, device=DEV)
        return {"case": c, "x": x, "logits": logits, "ids": i32(T, k), "w": torch.empty((T, k), device=DEV),
                "bufs": bufs, "ws": ws}
    if c["kind"] == "combine":
        y, p2r, w, sy = _combine_inputs(c, seed)
        return {"case": c, "y": y, "p2r": p2r, "w": w, "shared": sy,
                "out": torch.empty((c["T"], c["H"]), dtype=torch.bfloat16, device=DEV)}
    if c["kind"] == "reshard":
        g = _gen(seed)
        E, H, I, P = c["E"], c["H"], c["I"], c["P"]
        ep, tp = ((E // P, 2 * I, H), (E // P, H, I)), ((E, 2 * I // P, H), (E, H, I // P))
        s, d = (ep, tp) if c["dir"] == "ep_to_tp" else (tp, ep)
        src = [tuple(_normal(g, t, 0.02) for t in s) if not c["own"] or q == c["rank"] else (None, None)
               for q in range(P)]
        dst = tuple(torch.zeros(t, dtype=torch.bfloat16, device=DEV) for t in d)
        return {"case": c, "w13": [t[0] for t in src], "w2": [t[1] for t in src], "dst": dst}
    return {"case": c, **_kv_state(c, seed)}


def run(state):
    s, c = state, state["case"]
    if c["kind"] == "layer":
        layer = s["layer"]
        out = layer.forward(s["x"], s["logits"])
        return {"out": out, "topk_ids": layer.topk_ids, "topk_w": layer.topk_w}
    if c["kind"] == "ffn":
        return moe.grouped_ffn(s["x"], s["offsets"], s["w13"], s["w2"], y=s["y"], workspace=s["ws"])
    if c["kind"] == "dispatch":
        ids, w = moe.route(s["logits"], c["k"], s["ids"], s["w"])
        o = moe.permute(ids, c["E"], 0, c["E"], x=s["x"], out=s["bufs"], workspace=s["ws"])
        return {"topk_ids": ids, "topk_w": w, **o}
    if c["kind"] == "combine":
        return moe.combine(s["y"], s["p2r"], s["w"], out=s["out"], shared_y=s["shared"])
    if c["kind"] == "reshard":
        moe.reshard_experts(moe.EP_TO_TP if c["dir"] == "ep_to_tp" else moe.TP_TO_EP, c["rank"], c["E"], c["H"],
                            c["I"], s["w13"], s["w2"], *s["dst"])
        return s["dst"]
    moe.kv_slots(s["src_tab"], s["first"], c["page"], out=s["slot_src"])
    moe.kv_slots(s["dst_tab"], s["first"], c["page"], out=s["slot_dst"])
    dk, dv = s["dst"]
    for i in range(c["layers"]):
        if c["dir"] == "ep_to_tp":
            moe.kv_move([k[i] for k, _ in s["src"]], [v[i] for _, v in s["src"]], dk[i], dv[i], s["slot_src"],
                        s["slot_dst"], 0, 0, s["heads"], src_tokens=s["counts"])
        else:  # each TP rank's pool supplies its own heads
            for q, (k, v) in enumerate(s["src"]):
                moe.kv_move(k[i], v[i], dk[i], dv[i], s["slot_src"], s["slot_dst"], 0, q * s["heads"], s["heads"],
                            src_tokens=s["counts"][q])
    return {"k": dk, "v": dv, "slot_src": s["slot_src"], "slot_dst": s["slot_dst"]}


# ---------------------------------------------------------------- checking
def tolerance(case):
    # copies and slot vectors: the same bits
    if case["kind"] in ("reshard", "kv"):
        return "exact"
    # integers and copied rows the same; the gate weights are fp32
    if case["kind"] == "dispatch":
        return {"rel": 3e-7}  # measured 6e-8 off 64 bits
    # one rounding to bf16 (measured 1.7e-3 off 64 bits)
    if case["kind"] == "combine":
        return {"rel": 7e-3, "max": 2e-2}
    # bf16 outputs of fp32 sums over a bf16 intermediate (measured 2.9e-3)
    return {"rel": 1e-2, "max": 5e-2}


def _swiglu(x, w13, w2):
    """x [n, H] in 64 bits through one expert."""
    n = w2.shape[1]
    g = x @ w13[:n].double().t()
    u = x @ w13[n:].double().t()
    return (g * torch.sigmoid(g) * u) @ w2.double().t()


def _topk(logits, k):
    """Largest logits first, ties to the lower id; weights renormalised over the kept ones."""
    top = torch.sort(logits.double(), dim=1, descending=True, stable=True)
    return top.indices[:, :k], torch.softmax(top.values[:, :k], 1)


def exact(case, seed):
    c = case
    if c["kind"] == "layer":
        x, logits, w13, w2, sw13, sw2 = _layer_inputs(c, seed)
        ids, w = _topk(logits, c["k"])
        e0 = c["rank"] * w13.shape[0] if c["layout"] == "ep" else 0
        out = torch.zeros((c["T"], c["H"]), dtype=torch.float64, device=DEV)
        for e in range(w13.shape[0]):
            t, j = torch.nonzero(ids == e0 + e, as_tuple=True)
            if len(t):
                out.index_add_(0, t, w[t, j][:, None] * _swiglu(x[t].double(), w13[e], w2[e]))
        if c["shared"]:
            sb, sc = _shared_rows(c)
            out[sb:sb + sc] += _swiglu(x[sb:sb + sc].double(), sw13[0], sw2[0])
        return {"out": out, "topk_ids": ids.to(torch.int32), "topk_w": w}
    if c["kind"] == "ffn":
        x, off, w13, w2 = _ffn_inputs(c, seed)
        y = torch.zeros((c["n"], c["H"]), dtype=torch.float64, device=DEV)
        for e in range(c["El"]):
            a, b = int(off[e]), int(off[e + 1])
            if b > a:
                y[a:b] = _swiglu(x[a:b].double(), w13[e], w2[e])
        return y
    if c["kind"] == "dispatch":
        _, logits = _dispatch_inputs(c, seed)
        _, w = _topk(logits, c["k"])
        return {"topk_ids": None, "topk_w": w, "counts": None, "offsets": None, "row_to_pair": None,
                "pair_to_row": None, "x_perm": None}
    if c["kind"] == "combine":
        y, p2r, w, sy = _combine_inputs(c, seed)
        out = sy.double() if sy is not None else torch.zeros((c["T"], c["H"]), dtype=torch.float64, device=DEV)
        rows = p2r.reshape(c["T"], c["k"]).long()
        for j in range(c["k"]):
            out += w[:, j:j + 1].double() * y[rows[:, j]].double()
        return out
    return None
