"""Performance cases of the DAF library, through its public entry points.

A program that serves a request with this library selects the important tokens
(``daf_select_important``), recomputes the selection layers in full and every
later layer on the important and question rows only (``daf_decoder_layer``), or
brings its own projections and norms and calls the attention
(``daf_layer_attn``, or the stages one by one) and the row operations
(``daf_rmsnorm``, ``daf_linear``, ``daf_linear_swiglu``). A case is one such
call, or the few calls that such a program makes together, on inputs of the
Qwen2.5-7B widths (28 query heads, 4 KV heads, head_dim 128, hidden 3584, MLP
18944) unless it says otherwise.

A case is a dict of plain values: ``kind`` names the calls, ``L_d``, ``L_q`` and
``n`` list the requests of the batch (documents, question, important tokens,
separated by blanks), ``hq``, ``hkv``, ``d`` and ``dtype`` the attention shape.
"""
from __future__ import annotations

import math

import torch

import paper_2607_21599_amd as daf

HIDDEN, INTER, EPS, THETA = 3584, 18944, 1e-6, 1e6
QWEN = dict(hq=28, hkv=4, d=128, dtype="bf16")


def _case(kind, reqs, **kw):
    """reqs: (L_d, L_q, n) per request."""
    c = dict(kind=kind, L_d=" ".join(str(r[0]) for r in reqs), L_q=" ".join(str(r[1]) for r in reqs),
             n=" ".join(str(r[2]) for r in reqs))
    c.update(QWEN)
    c.update(kw)
    return c


def listed():
    batch8 = [(4096, 132, 614), (8192, 44, 1229), (12288, 140, 1843), (16384, 111, 2458), (20480, 167, 3072),
              (24576, 212, 3686), (28672, 64, 4301), (32768, 36, 4915)]
    cases = [
        # the smallest call: one fp32 layer of a tiny model over 4 documents of
        # 256 tokens; launches and latency are all of it
        ("layer_f32_1k", _case("layer", [(1024, 32, 154)], hq=4, hkv=1, d=64, dtype="f32")),
        # one layer's attention of a multi-hop question over 6 short documents
        ("layer_6k", _case("layer", [(6144, 64, 922)])),
        # the benchmark's layer: 32 documents of 1024 tokens
        ("layer_32k", _case("layer", [(32768, 128, 4915)])),
        # a serving batch: eight requests of 4k to 32k document tokens, ragged questions
        ("layer_batch8", _case("layer", batch8)),
        # the stages called one by one by a program that schedules them itself,
        # a large important set (r = 0.30)
        ("stages_16k_r30", _case("stages", [(16384, 128, 4915)])),
        # a short question over a long cache: stage 2 near the memory bound
        ("qdoc_32k_lq32", _case("qdoc", [(32768, 32, 0)])),
        # the scheme DAF is compared with: important and question rows over the whole context
        ("position_16k", _case("position", [(16384, 128, 2458)])),
        # the choice of the important tokens from the keys of three layers
        ("select_32k", _case("select", [(32768, 0, 4915)], layers=3)),
        # the MLP block of a program with its own layer loop: norm, gated
        # projections, down projection with the residual, ragged row count
        ("mlp_2586", _case("mlp", [(0, 2586, 0)], hidden=HIDDEN, inter=INTER)),
        # the first layer that recomputes only the important and question rows:
        # its compact state gathered from the full one, then the whole layer
        ("decoder_6k", _case("decoder", [(6144, 64, 922)], hidden=HIDDEN, inter=INTER)),
        ("decoder_32k", _case("decoder", [(32768, 128, 4915)], hidden=HIDDEN, inter=INTER)),
        # a selection layer: every row recomputed
        ("decoder_full_16k", _case("full", [(16384, 128, 0)], hidden=HIDDEN, inter=INTER)),
    ]
    return [dict(c, name=name) for name, c in cases]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: contexts of 512 to 128k document tokens, questions of 8
    to 256 tokens, r from 0.05 to 0.30, one request or a ragged batch, the
    head shapes of the tests, fp32 for the small layers."""
    while True:
        kind = rng.choice(["layer", "layer", "layer", "stages", "qdoc", "position", "select", "mlp", "decoder",
                           "decoder", "full"])
        kw = {}
        if kind in ("decoder", "full", "mlp"):
            kw.update(hidden=HIDDEN, inter=INTER)
        else:
            hq, hkv, d = rng.choice([(28, 4, 128), (28, 4, 128), (14, 2, 128), (8, 2, 64)])
            kw.update(hq=hq, hkv=hkv, d=d)
        hi = {"full": 16384, "position": 32768, "decoder": 65536}.get(kind, 131072)
        if kind in ("layer", "stages") and rng.random() < 0.2:
            kw.update(dtype="f32", hq=4, hkv=1, d=64)
            hi = 4096
        reqs = []
        for _ in range(rng.choice([1, 1, 1, 2, 4, 8]) if kind in ("layer", "stages", "qdoc", "select", "decoder") else 1):
            L_d = _log_int(rng, 512, hi)
            L_q = _log_int(rng, 8, 256)
            n = int(math.floor(rng.uniform(0.05, 0.30) * L_d + 0.5))
            if kind in ("qdoc", "full"):
                n = 0
            if kind == "select":
                L_q = 0
            if kind == "mlp":
                L_d, L_q, n = 0, _log_int(rng, 33, 16384), 0
            reqs.append((L_d, L_q, n))
        if kind == "select":
            kw["layers"] = rng.choice([1, 3, 3, 4])
        c = _case(kind, reqs, **kw)
        w, top = work(c), _LARGEST
        if w["flops"] <= top["flops"] and w["bytes"] <= top["bytes"]:
            return c


# ---- sizes and work ----------------------------------------------------------
def _reqs(c):
    return list(zip(*([int(x) for x in c[k].split()] for k in ("L_d", "L_q", "n"))))


def _attn_work(c):
    """FLOP and bytes of stage 1, stage 2 and the row movements around them."""
    eb = 2 if c["dtype"] == "bf16" else 4
    qrow, krow = c["hq"] * c["d"] * eb, c["hkv"] * c["d"] * eb
    per = 4 * c["d"] * c["hq"]
    f1 = f2 = b1 = b2 = bkv = bhid = bgat = 0
    for L_d, L_q, n in _reqs(c):
        f1 += per * n * (n + 1) // 2
        f2 += per * (L_q * L_d + L_q * (L_q + 1) // 2)
        b1 += 2 * n * (qrow + krow)
        b2 += 2 * (L_d + L_q) * krow + 2 * L_q * qrow
        bkv += 4 * (n + L_q) * krow
        bhid += (n + L_q) * qrow
        bgat += 2 * n * qrow
    return f1, f2, b1, b2, bkv, bhid, bgat


def work(c):
    f1, f2, b1, b2, bkv, bhid, bgat = _attn_work(c)
    kind, reqs = c["kind"], _reqs(c)
    if kind == "layer":  # the hidden rows are written beside the outputs
        return {"bytes": bgat + bkv + b1 + b2 + bhid, "flops": f1 + f2}
    if kind == "stages":  # the fusion reads the outputs again
        return {"bytes": bkv + b1 + b2 + 2 * bhid, "flops": f1 + f2}
    if kind == "qdoc":
        return {"bytes": b2, "flops": f2}
    if kind == "position":
        (L_d, L_q, n), = reqs
        # on average an important row sees half the documents
        pairs = n * (L_d + 1) // 2 + L_q * L_d + L_q * (L_q + 1) // 2
        return {"bytes": 2 * (L_d + L_q) * c["hkv"] * c["d"] * 2 + 2 * (n + L_q) * c["hq"] * c["d"] * 2,
                "flops": 4 * c["d"] * c["hq"] * pairs}
    if kind == "select":
        eb = 2 if c["dtype"] == "bf16" else 4
        rows = sum(r[0] for r in reqs)
        elems = c["layers"] * rows * c["hkv"] * c["d"]
        return {"bytes": 2 * elems * eb + 4 * rows + 4 * sum(r[2] for r in reqs), "flops": 3 * elems}
    H, I, QW, KW = c["hidden"], c["inter"], c["hq"] * c["d"], c["hkv"] * c["d"]
    if kind == "mlp":
        M = reqs[0][1]
        return {"bytes": 2 * (2 * M * H + 3 * H * I + H), "flops": 6 * M * H * I}
    rows = sum((r[2] if kind == "decoder" else r[0]) + r[1] for r in reqs)
    weights = H * (QW + 2 * KW) + QW * H + 3 * H * I
    flops = 2 * rows * weights
    bytes_ = 2 * weights + 4 * rows * H
    if kind == "decoder":
        bytes_ += bkv // 2 + sum(2 * (r[0] + r[1]) * KW * 2 for r in reqs)
        flops += f1 + f2
    else:
        flops += 4 * QW * sum((r[0] + r[1]) * (r[0] + r[1] + 1) // 2 for r in reqs)
    return {"bytes": bytes_, "flops": flops}


_LARGEST = {k: max(work(c)[k] for c in listed()) for k in ("bytes", "flops")}


# ---- inputs ------------------------------------------------------------------
def _cu(xs):
    out = [0]
    for x in xs:
        out.append(out[-1] + x)
    return out


def _batch(c):
    r = _reqs(c)
    return daf.Batch(_cu(x[0] for x in r), _cu(x[1] for x in r), _cu(x[2] for x in r))


def _cfg(c):
    return daf.AttnCfg(c["hq"], c["hkv"], c["d"], daf.DAF_BF16 if c["dtype"] == "bf16" else daf.DAF_F32)


def _inputs(c, seed):
    """The tensors of the case: projected q/k/v N(0, 1) * 0.5, the queries of
    each head scaled by 1 to 8 so that the heads range from a nearly uniform
    softmax to a peaked one; cached keys and values N(0, 1) * 0.5."""
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    dt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    hq, hkv, d, kind = c["hq"], c["hkv"], c["d"], c["kind"]
    reqs = _reqs(c)
    nd, nq, ni = (sum(r[i] for r in reqs) for i in range(3))
    s = {}

    def normal(*shape, std=0.5, dtype=dt):
        return torch.empty(shape, dtype=torch.float32, device="cuda").normal_(0.0, std, generator=g).to(dtype)

    head_scale = (8.0 ** (torch.arange(hq, device="cuda") / max(1, hq - 1)))[:, None]

    def queries(rows):
        return (normal(rows, hq, d, dtype=torch.float32) * head_scale).to(dt)

    idx = [torch.randperm(r[0], generator=g, device="cuda")[:r[2]].sort().values for r in reqs]
    s["idx"] = torch.cat(idx).to(torch.int32)
    if kind in ("layer", "stages", "position"):
        s["q_imp"], s["k_imp"], s["v_imp"] = queries(ni), normal(ni, hkv, d), normal(ni, hkv, d)
    if kind in ("layer", "stages", "qdoc", "position"):
        s["q_q"] = queries(nq)
        s["k_cache"], s["v_cache"] = normal(nd + nq, hkv, d), normal(nd + nq, hkv, d)
    if kind in ("layer", "stages"):
        s["k_q"], s["v_q"] = normal(nq, hkv, d), normal(nq, hkv, d)
        s["hidden"] = normal(nd + nq, hq * d)
    if kind == "position":
        (L_d, L_q, _), = reqs
        s["q"] = torch.cat([s["q_imp"], s["q_q"]])
        s["pos"] = torch.cat([s["idx"], torch.arange(L_d, L_d + L_q, dtype=torch.int32, device="cuda")])
    if kind == "select":
        # fresh keys deviate from the cached ones by noise of a per-token,
        # log-normal scale: a few tokens deviate much more than most
        scale = torch.empty((nd, 1, 1), device="cuda").normal_(0.0, 0.5, generator=g).exp() * 0.1
        cached = [normal(nd, hkv, d, dtype=torch.float32) for _ in range(c["layers"])]
        s["k_fresh"] = [(k + normal(nd, hkv, d, std=1.0, dtype=torch.float32) * scale).to(dt) for k in cached]
        s["k_cached"] = [k.to(dt) for k in cached]
    if kind in ("mlp", "decoder", "full"):
        H, I = c["hidden"], c["inter"]

        def weight(out, fan_in):
            return normal(out, fan_in, std=1.0 / math.sqrt(fan_in))

        def gain():
            return (1.0 + normal(H, std=0.1, dtype=torch.float32)).to(dt)

        s["w"] = {"w_post": gain(), "wgu": weight(2 * I, H), "wd": weight(H, I)}
        if kind == "mlp":
            s["x0"] = normal(nq, H, std=1.0)
        else:
            QW, KW = hq * d, hkv * d
            s["w"].update(w_in=gain(), wq=weight(QW, H), bq=normal(QW, std=0.1), wk=weight(KW, H),
                          bk=normal(KW, std=0.1), wv=weight(KW, H), bv=normal(KW, std=0.1), wo=weight(H, QW))
            s["x0"] = normal(nd + nq, H, std=1.0)
            pos = [torch.arange(r[0] + r[1], device="cuda") for r in reqs]
            if kind == "decoder":
                s["k_cache"], s["v_cache"] = normal(nd + nq, hkv, d), normal(nd + nq, hkv, d)
                tok = _cu(r[0] + r[1] for r in reqs)
                s["q_rows"] = torch.cat([torch.arange(t + r[0], t + r[0] + r[1], device="cuda") for t, r in zip(tok, reqs)])
                s["imp_rows"] = torch.cat([t + i for t, i in zip(tok, idx)])
                pos = idx + [torch.arange(r[0], r[0] + r[1], device="cuda") for r in reqs]
            s["pos"] = torch.cat(pos).to(torch.int32)
    return s


def prepare(c, seed):
    """The inputs, and the output buffers and workspace that a program keeps."""
    s = _inputs(c, seed)
    kind, hq, hkv, d = c["kind"], c["hq"], c["hkv"], c["d"]
    s["kind"], s["cfg"], s["batch"] = kind, _cfg(c), _batch(c)
    dt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    nd, nq, ni = (sum(r[i] for r in _reqs(c)) for i in range(3))

    def new(*shape, dtype=dt):
        return torch.zeros(shape, dtype=dtype, device="cuda")

    ws_bytes = 0
    if kind in ("layer", "stages", "qdoc"):
        s["o_imp"], s["o_q"] = new(ni, hq, d), new(nq, hq, d)
        s["lse_imp"], s["lse_q"] = new(hq, ni, dtype=torch.float32), new(hq, nq, dtype=torch.float32)
        size = daf.daf_layer_workspace_size if kind == "layer" else daf.daf_qdoc_workspace_size
        ws_bytes = size(s["cfg"], s["batch"])
        if kind == "layer":
            s["gathered"] = new(ni, hq * d)
            s["row_bytes"] = hq * d * s["hidden"].element_size()
    elif kind == "position":
        s["rows"], s["keys"] = s["q"].shape[0], s["k_cache"].shape[0]
        s["o"], s["lse"] = torch.zeros_like(s["q"]), new(hq, s["rows"], dtype=torch.float32)
    elif kind == "select":
        s["scores"], s["idx"] = new(nd, dtype=torch.float32), new(ni, dtype=torch.int32)
    elif kind == "mlp":
        M, H, I = nq, c["hidden"], c["inter"]
        s.update(M=M, H=H, I=I, h=new(M, H), m=new(M, I), y=new(M, H))
    else:
        H, I = c["hidden"], c["inter"]
        s["weights"] = daf.LayerWeights.from_tensors(s["w"], H, I, EPS, THETA)
        s["mode"] = daf.DAF_LAYER_DAF if kind == "decoder" else daf.DAF_LAYER_FULL
        s["x"] = new(ni + nq if kind == "decoder" else nd + nq, H)
        s["ni"], s["row_bytes"] = ni, H * 2
        ws_bytes = daf.daf_decoder_layer_workspace_size(s["cfg"], s["weights"], s["batch"], s["mode"])
    s["ws_bytes"] = ws_bytes
    s["ws"] = torch.empty(max(ws_bytes, 256), dtype=torch.uint8, device="cuda")
    return s


# ---- one pass ------------------------------------------------------------------
def run(s):
    kind, cfg, batch = s["kind"], s["cfg"], s["batch"]
    if kind == "layer":
        daf.daf_gather_important(batch, daf.DAF_SRC_TOKENS, s["hidden"], s["row_bytes"], s["idx"], s["gathered"])
        daf.daf_layer_attn(cfg, batch, s["idx"], s["q_imp"], s["k_imp"], s["v_imp"], s["q_q"], s["k_q"], s["v_q"],
                           s["k_cache"], s["v_cache"], s["o_imp"], s["lse_imp"], s["o_q"], s["lse_q"], s["hidden"],
                           s["ws"], s["ws_bytes"])
        names = ("gathered", "o_imp", "lse_imp", "o_q", "lse_q", "hidden", "k_cache", "v_cache")
        return {k: s[k] for k in names}
    if kind == "stages":
        daf.daf_fuse(cfg, batch, daf.DAF_FUSE_KV, s["idx"], k_imp=s["k_imp"], v_imp=s["v_imp"], k_q=s["k_q"],
                     v_q=s["v_q"], k_cache=s["k_cache"], v_cache=s["v_cache"])
        daf.daf_imp_self_attn(cfg, batch, s["q_imp"], s["k_imp"], s["v_imp"], s["o_imp"], s["lse_imp"])
        daf.daf_qdoc_attn(cfg, batch, s["q_q"], s["k_cache"], s["v_cache"], s["o_q"], s["lse_q"], s["ws"],
                          s["ws_bytes"])
        daf.daf_fuse(cfg, batch, daf.DAF_FUSE_HIDDEN, s["idx"], o_imp=s["o_imp"], o_q=s["o_q"], hidden=s["hidden"])
        return {k: s[k] for k in ("o_imp", "lse_imp", "o_q", "lse_q", "hidden", "k_cache", "v_cache")}
    if kind == "qdoc":
        daf.daf_qdoc_attn(cfg, batch, s["q_q"], s["k_cache"], s["v_cache"], s["o_q"], s["lse_q"], s["ws"],
                          s["ws_bytes"])
        return {"o_q": s["o_q"], "lse_q": s["lse_q"]}
    if kind == "position":
        daf.daf_position_attn(cfg, s["rows"], s["keys"], s["q"], s["pos"], s["k_cache"], s["v_cache"], s["o"],
                              s["lse"])
        return {"o": s["o"], "lse": s["lse"]}
    if kind == "select":
        daf.daf_select_important(cfg, batch, s["k_fresh"], s["k_cached"], s["scores"], s["idx"])
        return {"scores": s["scores"], "idx": s["idx"]}
    if kind == "mlp":
        daf.daf_rmsnorm(s["M"], s["H"], s["x0"], s["w"]["w_post"], EPS, s["h"])
        daf.daf_linear_swiglu(s["M"], s["I"], s["H"], s["h"], s["w"]["wgu"], s["m"])
        daf.daf_linear(s["M"], s["H"], s["I"], s["m"], s["w"]["wd"], None, s["x0"], s["y"])
        return {"h": s["h"], "m": s["m"], "y": s["y"]}
    if kind == "decoder":
        daf.daf_gather_important(batch, daf.DAF_SRC_TOKENS, s["x0"], s["row_bytes"], s["idx"], s["x"])
        torch.index_select(s["x0"], 0, s["q_rows"], out=s["x"][s["ni"]:])
        daf.daf_decoder_layer(cfg, s["weights"], batch, s["mode"], s["idx"], s["pos"], s["x"], s["k_cache"],
                              s["v_cache"], s["ws"], s["ws_bytes"])
        return {"x": s["x"], "k_cache": s["k_cache"], "v_cache": s["v_cache"]}
    # every row recomputed, from the embeddings that the program keeps
    s["x"].copy_(s["x0"])
    daf.daf_decoder_layer(cfg, s["weights"], batch, s["mode"], None, s["pos"], s["x"], None, None, s["ws"],
                          s["ws_bytes"])
    return {"x": s["x"]}


# ---- tolerances ------------------------------------------------------------------
def tolerance(c):
    if c["kind"] == "select":
        # fp32 sums of squares; one token traded for another of the same score
        # to rounding shifts the indices between the two
        return {"rel": 2e-6, "differ": 0.01}
    if c["dtype"] == "f32":
        return {"rel": 1e-5}
    # bf16 outputs: half an ulp each (2^-9 relative at most, 1.7e-3 in the
    # 2-norm), the probabilities or the intermediate activations rounded to
    # bf16 before the next product
    return {"rel": 1e-2}


# ---- the same in 64 bits -----------------------------------------------------------
def _attend(q, k, v, limit):
    """q [rows][Hq][D] over k, v [keys][Hkv][D] (64 bits), row i over keys
    0 .. limit[i] (ascending); outputs and LSE [Hq][rows]."""
    rows, hq, d = q.shape
    hkv = k.shape[1]
    o = torch.empty_like(q)
    lse = torch.empty((hq, rows), dtype=q.dtype, device=q.device)
    step = max(1, (1 << 25) // max(1, k.shape[0]))
    for h in range(hq):
        kh, vh = k[:, h * hkv // hq].contiguous(), v[:, h * hkv // hq].contiguous()
        for a in range(0, rows, step):
            lim = limit[a:a + step]
            end = int(lim[-1]) + 1
            sc = torch.mm(q[a:a + step, h].contiguous(), kh[:end].t().contiguous()).div_(math.sqrt(d))
            sc.masked_fill_(torch.arange(end, device=q.device)[None, :] > lim[:, None], -math.inf)
            l = torch.logsumexp(sc, 1)
            o[a:a + step, h] = torch.mm(sc.sub_(l[:, None]).exp_(), vh[:end])
            lse[h, a:a + step] = l
    return o, lse


def _stages(c, q_imp, k_imp, v_imp, q_q, k_cache, v_cache):
    """Both stages over the batch; k_cache and v_cache are the hybrid cache."""
    o1, l1, o2, l2 = [], [], [], []
    i0 = q0 = t0 = 0
    for L_d, L_q, n in _reqs(c):
        dev = q_q.device
        if n:
            o, l = _attend(q_imp[i0:i0 + n], k_imp[i0:i0 + n], v_imp[i0:i0 + n], torch.arange(n, device=dev))
            o1.append(o)
            l1.append(l)
        if L_q:
            o, l = _attend(q_q[q0:q0 + L_q], k_cache[t0:t0 + L_d + L_q], v_cache[t0:t0 + L_d + L_q],
                           torch.arange(L_d, L_d + L_q, device=dev))
            o2.append(o)
            l2.append(l)
        i0, q0, t0 = i0 + n, q0 + L_q, t0 + L_d + L_q
    return (torch.cat(o1) if o1 else None, torch.cat(l1, 1) if l1 else None, torch.cat(o2), torch.cat(l2, 1))


def _rows(c, idx):
    """Token rows of the important and of the question rows."""
    imp, qs, i0, t0 = [], [], 0, 0
    for L_d, L_q, n in _reqs(c):
        imp.append(t0 + idx[i0:i0 + n].long())
        qs.append(torch.arange(t0 + L_d, t0 + L_d + L_q, device=idx.device))
        i0, t0 = i0 + n, t0 + L_d + L_q
    return torch.cat(imp), torch.cat(qs)


def _norm(x, g):
    return x / torch.sqrt((x * x).mean(1, keepdim=True) + EPS) * g


def _rope(x, pos, d):
    half = d // 2
    ang = pos.double()[:, None] * THETA ** (-2.0 * torch.arange(half, device=x.device, dtype=torch.float64) / d)
    cs, sn = ang.cos()[:, None], ang.sin()[:, None]
    a, b = x[..., :half], x[..., half:]
    return torch.cat([a * cs - b * sn, b * cs + a * sn], -1)


def _mlp(h, wgu, wd, inter):
    g = torch.mm(h, wgu[:inter].t())
    m = g.div_(1.0 + torch.exp(-g)).mul_(torch.mm(h, wgu[inter:].t()))
    return m, torch.mm(m, wd.t())


def exact(c, seed):
    kind = c["kind"]
    if work(c)["flops"] > 1.2e13:
        return None
    s = _inputs(c, seed)
    f = lambda t: t.double()  # noqa: E731
    if kind in ("layer", "stages", "qdoc"):
        if kind == "qdoc":
            k, v = f(s["k_cache"]), f(s["v_cache"])
            q_imp = k_imp = v_imp = None
        else:
            q_imp, k_imp, v_imp = f(s["q_imp"]), f(s["k_imp"]), f(s["v_imp"])
            imp, qs = _rows(c, s["idx"])
            k, v = f(s["k_cache"]), f(s["v_cache"])
            k[imp], v[imp], k[qs], v[qs] = k_imp, v_imp, f(s["k_q"]), f(s["v_q"])
        o1, l1, o2, l2 = _stages(c, q_imp, k_imp, v_imp, f(s["q_q"]), k, v)
        if kind == "qdoc":
            return {"o_q": o2, "lse_q": l2}
        out = {"o_imp": o1, "lse_imp": l1, "o_q": o2, "lse_q": l2, "hidden": None, "k_cache": None, "v_cache": None}
        return dict(out, gathered=None) if kind == "layer" else out
    if kind == "position":
        o, l = _attend(f(s["q"]), f(s["k_cache"]), f(s["v_cache"]), s["pos"].long())
        return {"o": o, "lse": l}
    if kind == "select":
        dev = [(f(a) - f(b)).flatten(1).norm(dim=1) for a, b in zip(s["k_fresh"], s["k_cached"])]
        return {"scores": sum(dev) / len(dev), "idx": None}
    w = {k: f(t) for k, t in s["w"].items()}
    if kind == "mlp":
        x = f(s["x0"])
        h = _norm(x, w["w_post"])
        m, y = _mlp(h, w["wgu"], w["wd"], c["inter"])
        return {"h": h, "m": m, "y": x + y}
    d, hq, hkv, pos = c["d"], c["hq"], c["hkv"], s["pos"]
    x = f(s["x0"])
    if kind == "decoder":
        x = x[torch.cat([s["imp_rows"], s["q_rows"]])]
    h = _norm(x, w["w_in"])
    q = _rope((torch.mm(h, w["wq"].t()) + w["bq"]).view(-1, hq, d), pos, d)
    k = _rope((torch.mm(h, w["wk"].t()) + w["bk"]).view(-1, hkv, d), pos, d)
    v = (torch.mm(h, w["wv"].t()) + w["bv"]).view(-1, hkv, d)
    if kind == "decoder":
        ni = s["imp_rows"].shape[0]
        kc, vc = f(s["k_cache"]), f(s["v_cache"])
        rows = torch.cat([s["imp_rows"], s["q_rows"]])
        kc[rows], vc[rows] = k, v
        o1, _, o2, _ = _stages(c, q[:ni], k[:ni], v[:ni], q[ni:], kc, vc)
        o = torch.cat([o1, o2])
    else:
        (L_d, L_q, _), = _reqs(c)
        o, _ = _attend(q, k, v, torch.arange(L_d + L_q, device=q.device))
    x = x + torch.mm(o.reshape(-1, hq * d), w["wo"].t())
    x = x + _mlp(_norm(x, w["w_post"]), w["wgu"], w["wd"], c["inter"])[1]
    return {"x": x, "k_cache": kc, "v_cache": vc} if kind == "decoder" else {"x": x}
