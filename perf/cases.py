"""The decode work this library is used for, as timed and compared cases.

A case is one serving-stage call on one GPU: a contiguous operator range of a
block of decoder layers over a batch of sequences, through the package's
public entry points (tile_weights / DeviceBlock / DeviceBatch / DeviceState /
run_partition / attn_stage / ffn_stage / PartitionGraph). Layer shapes are the
ones the repository's workloads use (an 8B-shaped dense layer, a 4-layer
sliding-window hybrid block, a 64-expert top-8 MoE layer, a tensor-parallel
share, a tiny layer) plus a generic narrow layer with 64-wide heads.

Fields of a case: the layer shape (hidden, n_q, n_kv, head_dim, ffn or
n_experts / top_k / moe_ffn); n_layers, with window > 0 for every layer but
the last of a block of several; batch and the context range; part ("step":
the whole block, "attn" / "ffn": one stage of a one-layer block); layout of
the projection weights ("tiled", converted once, or "rows"); graph (the stage
captured once and replayed per step).
"""
import math

import numpy as np
import torch

from paper_2609_14237_amd import binding as B
from paper_2609_14237_amd import runtime as R

PAGE = B.PAGE_TOKENS


class _Cfg:
    """One layer's shape, as runtime.layer_cfg reads it."""

    def __init__(self, case, window):
        for k in ("hidden", "n_q", "n_kv", "head_dim", "ffn", "n_experts", "top_k", "moe_ffn"):
            setattr(self, k, case[k])
        self.window = window
        self.rope_theta, self.rms_eps = 10000.0, 1e-6


def _cfgs(case):
    n = case["n_layers"]
    return [_Cfg(case, case["window"] if n > 1 and l < n - 1 else 0) for l in range(n)]


def _dense(ffn=14336, n_q=32, n_kv=8, head_dim=128, hidden=4096):
    return dict(hidden=hidden, n_q=n_q, n_kv=n_kv, head_dim=head_dim, ffn=ffn, n_experts=0, top_k=0, moe_ffn=0,
                n_layers=1, window=0)


def _moe():
    return dict(hidden=4096, n_q=32, n_kv=4, head_dim=128, ffn=0, n_experts=64, top_k=8, moe_ffn=1536,
                n_layers=1, window=0)


def _case(shape, batch, ctx_lo, ctx_hi, part, layout, graph=False, **more):
    return dict(shape, batch=batch, ctx_lo=ctx_lo, ctx_hi=ctx_hi, part=part, layout=layout, graph=graph, **more)


def listed():
    d8 = _dense()
    return [
        # The smallest call: a tiny layer (FFN width 688 has no tiled form), all latency and launches.
        _case(_dense(ffn=688, n_q=4, n_kv=2, head_dim=64, hidden=256), 4, 128, 128, "step", "rows", name="tiny_step"),
        # One interactive request on the 8B-shaped layer, replayed as a graph: the latency of a single token.
        _case(d8, 1, 3000, 3000, "step", "tiled", True, name="dense8b_b1_step"),
        # A handful of requests, an odd number of them with ragged contexts: light serving load.
        _case(d8, 13, 512, 4096, "step", "tiled", name="dense8b_b13_step"),
        # Ordinary serving load: batch 64, ragged contexts, the whole layer.
        _case(d8, 64, 512, 4096, "step", "tiled", name="dense8b_b64_step"),
        # A narrow layer with 64-wide heads on untouched row-major weights, ragged batch of 100 short chats.
        _case(_dense(ffn=8192, n_q=32, n_kv=8, head_dim=64, hidden=2048), 100, 64, 2048, "step", "rows",
              name="narrow_rows_b100_step"),
        # The attention worker of a disaggregated deployment at high load (the benchmark's batch and context).
        _case(d8, 256, 8192, 8192, "attn", "tiled", name="dense8b_b256_attn"),
        # The FFN worker at the same load.
        _case(d8, 256, 16, 16, "ffn", "tiled", name="dense8b_b256_ffn"),
        # An FFN worker gathering the requests of many attention workers: the top of the FFN batch sweep.
        _case(d8, 2048, 16, 16, "ffn", "tiled", name="dense8b_b2048_ffn"),
        # Hybrid block: three sliding-window layers on page rings, then a full layer, long ragged contexts.
        _case(dict(d8, n_layers=4, window=1024), 128, 1024, 32768, "step", "tiled", name="hybrid4_b128_step"),
        # The expert stage of the MoE layer at high load: every expert busy.
        _case(_moe(), 512, 16, 16, "ffn", "tiled", name="moe_b512_ffn"),
        # The MoE layer at light load: few rows per expert.
        _case(_moe(), 24, 2048, 16384, "step", "tiled", name="moe_b24_step"),
        # One GPU's share of the 8B-shaped layer under 8-way tensor parallelism, batch 256.
        _case(_dense(ffn=1792, n_q=4, n_kv=1), 256, 8192, 8192, "step", "tiled", name="tp8_b256_step"),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _cost(case):
    """Rough seconds of a pass, to keep drawn cases below the largest listed one."""
    w = work(case)
    return w["bytes"] / 6e12 + w["flops"] / 1e15


def draw(rng):
    while True:
        kind = rng.choice(["dense_step", "dense_step", "attn", "ffn", "ffn", "narrow", "hybrid", "moe_ffn", "moe_step",
                           "share"])
        layout = rng.choice(["tiled", "tiled", "rows"])
        graph = rng.random() < 0.25
        hi = _log_int(rng, 64, 32768)
        lo = max(1, int(hi * rng.uniform(0.05, 1.0)))
        if kind == "dense_step":
            c = _case(_dense(), _log_int(rng, 1, 384), lo, hi, "step", layout, graph)
        elif kind == "attn":
            c = _case(_dense(n_kv=rng.choice([4, 8])), _log_int(rng, 1, 512), lo, hi, "attn", layout, graph)
        elif kind == "ffn":
            c = _case(_dense(), _log_int(rng, 1, 2048), PAGE, PAGE, "ffn", layout, graph)
        elif kind == "narrow":
            hidden = rng.choice([256, 520, 1024, 2048])
            n_kv = rng.choice([2, 4, 8])
            c = _case(_dense(ffn=rng.choice([688, 1376, 2816, 8192]), n_q=n_kv * rng.choice([1, 2, 4]), n_kv=n_kv,
                             head_dim=64, hidden=hidden), _log_int(rng, 1, 300), lo, hi, "step", "rows", graph)
        elif kind == "hybrid":
            c = _case(dict(_dense(), n_layers=rng.choice([2, 3, 4]), window=rng.choice([512, 1000, 1024, 2048])),
                      _log_int(rng, 1, 160), lo, hi, "step", layout, graph)
        elif kind == "moe_ffn":
            c = _case(_moe(), _log_int(rng, 1, 1024), PAGE, PAGE, "ffn", layout, graph)
        elif kind == "moe_step":
            c = _case(_moe(), _log_int(rng, 1, 512), lo, hi, "step", layout, graph)
        else:
            tp = rng.choice([2, 4, 8])
            c = _case(_dense(ffn=14336 // tp, n_q=32 // tp, n_kv=8 // tp), _log_int(rng, 1, 512), lo, hi, "step",
                      layout, graph)
        tokens = c["batch"] * (lo + hi) / 2 if c["part"] != "ffn" else 0
        if tokens * c["n_kv"] * c["head_dim"] * 4 > 9e9:  # one pool below the listed ones
            continue
        if _cost(c) <= max(_cost(x) for x in listed()):
            return c


# ---------------------------------------------------------------- inputs

def _gen(seed, *idx):
    h = 0x243F6A8885A308D3 ^ (seed * 0x9E3779B97F4A7C15)
    for i in idx:
        h = (h * 0x100000001B3 + i + 1) & ((1 << 63) - 1)
    g = torch.Generator(device="cuda")
    g.manual_seed(h & ((1 << 63) - 1))
    return g


def _normal(shape, g, std, mean=0.0):
    return torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(mean, std, generator=g)


def _contexts(case, seed):
    r = np.random.RandomState(seed % (1 << 31))
    return r.randint(case["ctx_lo"], case["ctx_hi"] + 1, case["batch"]).astype(np.int32)


def _weights(cfg, seed, layer):
    H, qkv = cfg.hidden, (cfg.n_q + 2 * cfg.n_kv) * cfg.head_dim
    n = lambda j, shape, std, mean=0.0: _normal(shape, _gen(seed, 1, layer, j), std, mean)  # noqa: E731
    w = {"g_attn": n(0, (H,), 0.02, 1.0), "w_qkv": n(1, (qkv, H), 0.02), "w_o": n(2, (H, cfg.n_q * cfg.head_dim), 0.02),
         "g_ffn": n(3, (H,), 0.02, 1.0)}
    if cfg.n_experts:
        E, I = cfg.n_experts, cfg.moe_ffn
        w.update(w_router=n(4, (E, H), H ** -0.5), w_gate_up=n(5, (E, 2 * I, H), 0.02), w_down=n(6, (E, H, I), 0.02))
    else:
        w.update(w_gate_up=n(5, (2 * cfg.ffn, H), 0.02), w_down=n(6, (H, cfg.ffn), 0.02))
    return w


def _ffn_weights_only(w):
    return {k: v for k, v in w.items() if k not in ("w_qkv", "w_o", "g_attn")}


def _attn_weights_only(w):
    return {k: v for k, v in w.items() if k in ("w_qkv", "w_o", "g_attn")}


def _x(case, seed):
    # Residual stream: small, as after the first layers, so that the stage's own result is most of the output;
    # unit size before an expert layer, as deep in a stack.
    return _normal((case["batch"], case["hidden"]), _gen(seed, 3), 1.0 if case["n_experts"] else 0.25)


def _alloc(pages, ctx, cols, seed):
    table = np.zeros((len(ctx), cols), np.int32)
    st = B.ods_kv_alloc(pages, ctx, len(ctx), seed, cols, table)
    assert st == B.ODS_OK, B.ods_last_error()
    return table


def _inputs(case, seed):
    """Host contexts and tables, device weights and KV pools."""
    cfgs = _cfgs(case)
    ctx = _contexts(case, seed)
    need = -(-ctx.astype(np.int64) // PAGE)
    inp = {"cfgs": cfgs, "ctx": ctx, "x": _x(case, seed)}
    inp["weights"] = [_weights(c, seed, l) for l, c in enumerate(cfgs)]
    inp["cols"] = int(need.max())
    inp["table"] = np.zeros((case["batch"], inp["cols"]), np.int32)
    inp["ring"], inp["pools"], inp["pages"] = None, [None] * len(cfgs), [0] * len(cfgs)
    if case["part"] == "ffn":
        return inp
    # A returned pool is the same size whatever the contexts drawn; a large one holds what they need and some slack.
    pages = -(-case["ctx_hi"] // PAGE) * case["batch"] if _returns_pool(case) else int(need.sum()) * 9 // 8 + 1
    inp["table"] = _alloc(pages, ctx, inp["cols"], seed)
    windows = [c.window for c in cfgs if c.window]
    ring_pages = 0
    if windows:
        cols = -(-max(windows) // PAGE) + 1
        held = np.minimum(ctx, cols * PAGE).astype(np.int32)
        ring_pages = case["batch"] * cols
        inp["ring"] = _alloc(ring_pages, held, cols, seed + 1)
    for l, c in enumerate(cfgs):
        n = ring_pages if c.window else pages
        pool = torch.empty((n, 2, c.n_kv, PAGE * c.head_dim), dtype=torch.bfloat16, device="cuda")
        pool.normal_(0.0, 1.0, generator=_gen(seed, 2, l))
        pool[:, 0].mul_(1.75)  # keys large enough that attention concentrates on some tokens, as it does in use
        inp["pools"][l], inp["pages"][l] = pool, n
    return inp


def _returns_pool(case):
    """Whether the pass returns the KV pools (its updated state): where they are of moderate size."""
    if case["part"] == "ffn":
        return False
    tokens = case["batch"] * (case["ctx_lo"] + case["ctx_hi"]) / 2
    return case["n_layers"] == 1 and tokens * 2 * case["n_kv"] * case["head_dim"] <= 1.2e8


def prepare(case, seed):
    inp = _inputs(case, seed)
    tiled = case["layout"] == "tiled"
    weights = []
    for cfg, w in zip(inp["cfgs"], inp["weights"]):
        w = R.tile_weights(cfg, w) if tiled else w
        if case["part"] == "ffn":
            w = _ffn_weights_only(w)
        elif case["part"] == "attn":
            w = _attn_weights_only(w)
        weights.append(w)
    inp["weights"] = None
    block = R.DeviceBlock(inp["cfgs"], weights, inp["pools"], inp["pages"], pretiled=tiled)
    ring = None if inp["ring"] is None else torch.from_numpy(inp["ring"]).cuda()
    batch = R.DeviceBatch(torch.from_numpy(inp["ctx"]).cuda(), torch.from_numpy(inp["table"]).cuda(), ring_table=ring)
    state = R.DeviceState(block, batch)
    resid = state.view("resid", case["batch"], case["hidden"])
    n_ops = block.num_ops()
    lo, hi = {"step": (0, n_ops), "attn": (0, 6), "ffn": (6, n_ops)}[case["part"]]
    resid.copy_(inp["x"])
    graph = R.PartitionGraph(block, lo, hi, batch, state) if case["graph"] else None
    pools = [p for p in inp["pools"] if p is not None] if _returns_pool(case) else []
    return {"part": case["part"], "block": block, "batch": batch, "state": state, "resid": resid, "x": inp["x"],
            "range": (lo, hi), "graph": graph, "pools": pools, "pool_refs": inp["pools"]}


def run(s):
    s["resid"].copy_(s["x"])  # the activations this step starts from arrive in the stage's bound buffer
    if s["graph"] is not None:
        s["graph"].launch()
    elif s["part"] == "attn":
        R.attn_stage(s["block"], 0, s["batch"], s["state"])
    elif s["part"] == "ffn":
        R.ffn_stage(s["block"], 0, s["batch"], s["state"])
    else:
        R.run_partition(s["block"], s["range"][0], s["range"][1], s["batch"], s["state"])
    return {"resid": s["resid"], "pools": s["pools"]}


def work(case):
    cfgs = _cfgs(case)
    Bn, H, d = case["batch"], case["hidden"], case["head_dim"]
    mean_ctx = (case["ctx_lo"] + case["ctx_hi"]) / 2
    nbytes, flops = 2.0 * 2 * Bn * H, 0.0  # residual in and out
    for c in cfgs:
        if case["part"] != "ffn":
            qkv, q = (c.n_q + 2 * c.n_kv) * d, c.n_q * d
            span = min(mean_ctx, c.window) if c.window else mean_ctx
            nbytes += 2.0 * (H * qkv + H * q) + Bn * span * c.n_kv * d * 4.0 + Bn * c.n_kv * d * 4.0
            flops += 2.0 * Bn * (H * qkv + H * q) + 4.0 * Bn * span * c.n_q * d
        if case["part"] != "attn":
            if c.n_experts:
                E, k, I = c.n_experts, c.top_k, c.moe_ffn
                busy = E * (1.0 - (1.0 - k / E) ** Bn)
                nbytes += 2.0 * (E * H + busy * 3 * I * H)
                flops += 2.0 * Bn * (E * H + k * 3 * I * H)
            else:
                nbytes += 2.0 * 3 * H * c.ffn
                flops += 2.0 * Bn * 3 * H * c.ffn
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # bf16 live buffers between operators: about three to four times the distance from 64 bits measured at the listed
    # cases (one stage 0.0033, one layer up to 0.0068, the four-layer block 0.013). Where a router logit moves past a
    # near tie a token takes another expert, a large difference on few rows (0.01 in all against 64 bits).
    if case["n_experts"]:
        return {"rel": 3e-2, "max": 0.99}
    if case["n_layers"] > 1:
        return {"rel": 3e-2}
    return {"rel": 2e-2 if case["part"] == "step" else 1e-2}


# ---------------------------------------------------------------- the same in 64 bits

def _rope(u, pos, theta):
    half = u.shape[-1] // 2
    inv = theta ** (-2.0 * torch.arange(half, dtype=torch.float64, device=u.device) / u.shape[-1])
    ang = (pos.double()[:, None] * inv)[:, None, :]
    c, s = torch.cos(ang), torch.sin(ang)
    a, b = u[..., :half], u[..., half:]
    return torch.cat([a * c - b * s, b * c + a * s], dim=-1)


def _norm(x, gain, eps):
    return x * torch.rsqrt((x * x).mean(-1, keepdim=True) + eps) * gain.double()


def _attention(cfg, w, pool, inp, x, ring, kept):
    """Attention stage in 64 bits; kept: the pool in 64 bits with the new tokens' keys and values, or None."""
    Bn, d, g = x.shape[0], cfg.head_dim, cfg.n_q // cfg.n_kv
    ctx = inp["ctx"]
    qkv = _norm(x, w["g_attn"], cfg.rms_eps) @ w["w_qkv"].double().T
    qkv = qkv.view(Bn, cfg.n_q + 2 * cfg.n_kv, d)
    pos = torch.from_numpy(ctx.astype(np.int64) - 1).to(x.device)
    q = _rope(qkv[:, : cfg.n_q], pos, cfg.rope_theta)
    k = _rope(qkv[:, cfg.n_q: cfg.n_q + cfg.n_kv], pos, cfg.rope_theta)
    v = qkv[:, cfg.n_q + cfg.n_kv:]
    o = torch.empty((Bn, cfg.n_kv, g, d), dtype=torch.float64, device=x.device)
    for b in range(Bn):
        p = int(ctx[b]) - 1
        lo = max(0, p - cfg.window + 1) if cfg.window else 0
        lp = np.arange(lo // PAGE, p // PAGE + 1)
        table = inp["ring"] if ring else inp["table"]
        ids = torch.from_numpy(table[b, lp % table.shape[1] if ring else lp].astype(np.int64)).to(x.device)
        blk = pool[ids].double()
        K = blk[:, 0].view(len(lp), cfg.n_kv, PAGE, d).permute(1, 0, 2, 3).reshape(cfg.n_kv, -1, d)
        V = blk[:, 1].view(len(lp), cfg.n_kv, d, PAGE).permute(1, 0, 3, 2).reshape(cfg.n_kv, -1, d)
        t0, t1 = lo - int(lp[0]) * PAGE, p - int(lp[0]) * PAGE
        K, V = K[:, t0: t1 + 1].contiguous(), V[:, t0: t1 + 1].contiguous()
        K[:, -1], V[:, -1] = k[b], v[b]
        s = torch.bmm(q[b].view(cfg.n_kv, g, d), K.transpose(1, 2).contiguous()) / math.sqrt(d)
        o[b] = torch.bmm(torch.softmax(s, -1), V)
        if kept is not None:
            page, slot = int(ids[-1]), p % PAGE
            kept.view(kept.shape[0], 2, cfg.n_kv, PAGE, d)[page, 0, :, slot] = k[b]
            kept.view(kept.shape[0], 2, cfg.n_kv, d, PAGE)[page, 1, :, :, slot] = v[b]
    return x + o.reshape(Bn, -1) @ w["w_o"].double().T


def _ffn(cfg, w, x):
    hn = _norm(x, w["g_ffn"], cfg.rms_eps)
    if not cfg.n_experts:
        gu = hn @ w["w_gate_up"].double().T
        act = torch.nn.functional.silu(gu[:, : cfg.ffn]) * gu[:, cfg.ffn:]
        return x + act @ w["w_down"].double().T
    z, ids = torch.topk(hn @ w["w_router"].double().T, cfg.top_k, dim=-1)
    p = torch.softmax(z, -1)
    out = x.clone()
    for e in range(cfg.n_experts):
        rows, slot = torch.nonzero(ids == e, as_tuple=True)
        if rows.numel():
            gu = hn[rows] @ w["w_gate_up"][e].double().T
            act = torch.nn.functional.silu(gu[:, : cfg.moe_ffn]) * gu[:, cfg.moe_ffn:]
            out[rows] += p[rows, slot, None] * (act @ w["w_down"][e].double().T)
    return out


def exact(case, seed):
    inp = _inputs(case, seed)
    x = inp["x"].double()
    pools = []
    for l, cfg in enumerate(inp["cfgs"]):
        w = inp["weights"][l]
        if case["part"] != "ffn":
            kept = inp["pools"][l].double() if _returns_pool(case) else None
            x = _attention(cfg, w, inp["pools"][l], inp, x, cfg.window > 0, kept)
            if kept is not None:
                pools.append(kept)
        if case["part"] != "attn":
            x = _ffn(cfg, w, x)
    return {"resid": x, "pools": pools}
