"""The measured cases: what a program that uses this library has it do.

A case is one layer's call of the routed sparse-attention path at one shape.
Its `kind` says which calls one pass makes, its other fields are the shape,
the dtype and the selection rule (`vsa2_problem`, `vsa2_select`):

  path     pool, route, inference forward: one serving call of the operation
  op       one training step of the whole operation: pool, route, forward,
           coarse branch and gated merge, and all their gradients
  route    pool and route with the transposed lists (the router alone)
  forward  inference forward over given block lists
  train    training forward and backward over given block lists
  coarse   the coarse branch alone: MeanPool_B, dense attention among the
           cube means, gated merge, and their gradients

Sizes are those of the workloads in `workload.py` (grids 8x16x16 to
40x48x80, 2 to 40 heads, D = 64 and 128, top-k, mass and per-sequence
selection) with the head count reduced where the full one only repeats work,
and odd, padded and text-joined grids as in the tests.  Inputs follow the
recipe of `workload.py` (cube mean + 0.5 noise, log-normal cube norms when
`skewed`), drawn on the GPU.
"""
import math

import torch

import paper_2609_32882_amd as vsa2

B = 64                      # tokens per 4x4x4 cube
TOPK, MASS, SEQ = vsa2.VSA2_SEL_TOPK, vsa2.VSA2_SEL_MASS, vsa2.VSA2_SEL_SEQ_TOPK


def _case(kind, t, h, w, hq, hkv, d=128, batch=1, dtype="bf16", rt=2, rh=2, rw=2, mode=TOPK, k=0, mass=0.0,
          cap=0, text=0, skewed=False, **kw):
    return dict(kind=kind, batch=batch, hq=hq, hkv=hkv, d=d, t=t, h=h, w=w, rt=rt, rh=rh, rw=rw, dtype=dtype,
                mode=mode, k=k, mass=mass, cap=cap, text=text, skewed=skewed, **kw)


def listed():
    return [
        # the smallest call (the "tiny" workload, fp32): launches and host time count
        _case("path", 8, 16, 16, 2, 2, d=64, dtype="f32", k=8, name="path-tiny-f32"),
        # one training step of the whole operation in a 480p model's layer
        _case("op", 20, 32, 56, 12, 12, k=70, name="op-480p"),
        # the router of a 720p layer
        _case("route", 20, 48, 80, 40, 40, k=120, name="route-720p"),
        # mass selection on the 720p latent grid itself (padded, uneven norms), grouped heads
        _case("route", 21, 45, 80, 10, 2, mode=MASS, mass=0.9, cap=240, skewed=True, name="route-mass-latent"),
        # the paper's per-sequence rule on a long clip, grouped heads
        _case("route", 40, 48, 80, 10, 2, mode=SEQ, k=120, name="route-seq-long"),
        # VSA's cube-level router (R = B): small score maps, so selection and list building count
        _case("route", 20, 48, 80, 40, 40, rt=4, rh=4, rw=4, k=120, name="route-vsa-720p"),
        # serving forward of a 480p and of a 720p layer
        _case("forward", 20, 32, 56, 12, 12, k=70, name="forward-480p"),
        _case("forward", 20, 48, 80, 40, 40, k=120, name="forward-720p"),
        # a small odd-sized training call: batch 2, D = 64, every axis cut
        _case("train", 7, 13, 22, 4, 2, d=64, batch=2, k=6, name="train-small-d64"),
        # the benchmark's training step (720p, 40 heads, top-120)
        _case("train", 20, 48, 80, 40, 40, k=120, name="train-720p"),
        # log-normal cube norms with mass selection and a ragged text tail: uneven lists, large magnitudes
        _case("train", 20, 32, 56, 12, 6, mode=MASS, mass=0.9, cap=140, text=200, skewed=True,
              name="train-mass-text"),
        # the coarse branch and gated merge beside a 720p layer
        _case("coarse", 20, 48, 80, 40, 40, name="coarse-720p"),
    ]


# --------------------------------------------------------------------------
# shapes
# --------------------------------------------------------------------------
def _cubes(c):
    return -(-c["t"] // 4) * -(-c["h"] // 4) * -(-c["w"] // 4)


def _blocks(c):
    return _cubes(c) + -(-c["text"] // B)


def _pooled(c):
    return (4 // c["rt"]) * (4 // c["rh"]) * (4 // c["rw"])


def _per_row(c):
    """Video blocks kept per row (the cap under mass selection)."""
    return min(c["cap"] if c["mode"] == MASS else c["k"], _cubes(c))


def _kept(c):
    """Video blocks a row keeps on average.  Mass selection on these inputs:
    scaled scores are about N(0, 1), so a mass of 0.9 (0.5) takes the best 61%
    (16%) of a row's blocks; log-normal norms peak the rows (3% and 1%, as
    counted on the 720p grid); never more than the cap."""
    if c["mode"] != MASS:
        return _per_row(c)
    share = (0.03 if c["mass"] > 0.7 else 0.01) if c["skewed"] else (0.61 if c["mass"] > 0.7 else 0.16)
    return max(1, min(_per_row(c), int(share * _cubes(c))))


def _pairs(c, kept=None):
    """Block pairs of the attention: `kept` video blocks a row (default: the
    most that the rule allows), and the text blocks in full."""
    n, m = _cubes(c), _blocks(c) - _cubes(c)
    return c["batch"] * c["hq"] * (n * ((_per_row(c) if kept is None else kept) + m) + m * (n + m))


def _size(c):
    return 2 if c["dtype"] == "bf16" else 4


def _tdtype(c):
    return torch.bfloat16 if c["dtype"] == "bf16" else torch.float32


def _problem(c):
    return vsa2.make_problem(c["batch"], c["hq"], c["hkv"], c["d"], c["t"], c["h"], c["w"], Rt=c["rt"], Rh=c["rh"],
                             Rw=c["rw"], dtype=vsa2.VSA2_BF16 if c["dtype"] == "bf16" else vsa2.VSA2_F32,
                             text_len=c["text"])


def _select(c):
    return vsa2.vsa2_select(c["mode"], c["k"], c["mass"], c["cap"])


# --------------------------------------------------------------------------
# draws
# --------------------------------------------------------------------------
# MFMA time of a case in "bf16 block pairs" (fp32 runs at about 1/16 of the
# bf16 rate): the drawn ones stay below the listed maximum
_MOST = 40 * 1200 * 120 * 3.5


def _cost(c):
    rate = 1 if c["dtype"] == "bf16" else 16
    n, g = _cubes(c), _pooled(c)
    route = c["batch"] * c["hq"] * (n * g / 64.0) ** 2
    fine = _pairs(c) if c["kind"] in ("path", "op", "forward", "train") else 0
    grad = 3.5 if c["kind"] in ("op", "train") else 1
    return rate * (fine * grad + (route if c["kind"] in ("path", "op", "route") else 0)) * c["d"] / 128.0


def draw(rng):
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    while True:
        kind = rng.choice(("path", "op", "route", "forward", "train", "coarse"))
        t, h, w = log(4, 40), log(12, 48), log(12, 80)
        grp = rng.choice((1, 1, 1, 2, 4, 5))
        hkv = max(1, log(1, 40) // grp)
        rt, rh, rw = rng.choice(((2, 2, 2), (2, 2, 2), (2, 2, 2), (4, 4, 4), (2, 2, 4), (2, 4, 4)))
        mode = rng.choice((TOPK, TOPK, MASS, SEQ) if kind == "route" else (TOPK, TOPK, MASS))
        c = _case(kind, t, h, w, hkv * grp, hkv, d=rng.choice((64, 128, 128)), batch=rng.choice((1, 1, 2)),
                  dtype=rng.choice(("bf16", "bf16", "bf16", "f32")), rt=rt, rh=rh, rw=rw, mode=mode,
                  text=log(1, 512) if kind in ("forward", "train") and rng.random() < 0.3 else 0,
                  skewed=rng.random() < 0.3)
        n = _cubes(c)
        keep = max(1, min(n, int(n * rng.uniform(0.05, 0.25))))
        if kind == "coarse":
            c["mode"], c["k"] = TOPK, keep      # unused by the coarse branch
        elif mode == MASS:
            c["mass"], c["cap"] = rng.choice((0.5, 0.9)), keep
        else:
            c["k"] = keep
        tokens = c["batch"] * c["hq"] * _blocks(c) * B
        if (_cost(c) <= _MOST and tokens <= 40 * 76800 and n <= 2400
                and c["batch"] * c["hq"] * n * n <= 40 * 1440 * 1440):
            return c


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------
def _real(c, dev):
    """bool [joint tokens]: token is not padding (grid or text tail)."""
    nt, nh, nw = -(-c["t"] // 4), -(-c["h"] // 4), -(-c["w"] // 4)
    a = torch.arange(4, device=dev)
    ok = [(torch.arange(m, device=dev)[:, None] * 4 + a < s) for m, s in ((nt, c["t"]), (nh, c["h"]), (nw, c["w"]))]
    v = (ok[0][:, None, None, :, None, None] & ok[1][None, :, None, None, :, None]
         & ok[2][None, None, :, None, None, :]).reshape(-1)
    m = _blocks(c) - _cubes(c)
    return torch.cat([v, torch.arange(m * B, device=dev) < c["text"]])


def _tokens(c, gen, heads, mean=True):
    """[batch, heads, joint tokens, d]: the recipe of the workloads."""
    dev = "cuda"
    n, m, d = _cubes(c), _blocks(c) - _cubes(c), c["d"]
    x = torch.randn((c["batch"], heads, n + m, B, d), generator=gen, device=dev)
    if mean:
        mu = torch.randn((c["batch"], heads, n, 1, d), generator=gen, device=dev)
        if c["skewed"]:
            mu *= torch.randn((c["batch"], heads, n, 1, 1), generator=gen, device=dev).exp()
        x[:, :, :n].mul_(0.5).add_(mu)
    x = x.reshape(c["batch"], heads, (n + m) * B, d)
    x *= _real(c, dev)[:, None]                 # padding tokens hold zeros
    return x.to(_tdtype(c))


def _mask(c, q, k):
    """bool [batch, hq, blocks, blocks]: a selection by the cube means' scores
    (what the router picks on these inputs), text blocks joined in full."""
    n, m, d = _cubes(c), _blocks(c) - _cubes(c), c["d"]
    cnt = _real(c, q.device)[:n * B].reshape(n, B).sum(1).float()[:, None]
    qc = q[:, :, :n * B].reshape(c["batch"], c["hq"], n, B, d).float().sum(3) / cnt
    kc = k[:, :, :n * B].reshape(c["batch"], c["hkv"], n, B, d).float().sum(3) / cnt
    keep = torch.zeros((c["batch"], c["hq"], n + m, n + m), dtype=torch.bool, device=q.device)
    for b in range(c["batch"]):
        for h in range(c["hq"]):
            p = torch.softmax(qc[b, h] @ kc[b, h // (c["hq"] // c["hkv"])].t().contiguous() / math.sqrt(d), -1)
            p, idx = torch.sort(p, dim=-1, descending=True, stable=True)
            if c["mode"] == MASS:
                full = torch.cumsum(p.double(), -1) - p.double() < c["mass"]
                take = full & (torch.arange(n, device=q.device) < c["cap"])
            else:
                take = (torch.arange(n, device=q.device) < c["k"]).expand(n, n)
            keep[b, h, :n, :n].scatter_(1, idx, take)
    keep[:, :, n:, :] = True
    keep[:, :, :, n:] = True
    return keep


def _lists(c, keep):
    """CSR of the mask and its transpose, as route() and joint_lists() lay them out."""
    nb, grp = _blocks(c), c["hq"] // c["hkv"]

    def ptr(x):
        return torch.cat([x.new_zeros(1), x.cumsum(0)]).to(torch.int32)

    rows = keep.reshape(-1, nb)
    cols = keep.reshape(c["batch"], c["hkv"], grp * nb, nb).transpose(2, 3).reshape(-1, grp * nb)
    return dict(row_ptr=ptr(rows.sum(1)), col_idx=rows.nonzero()[:, 1].to(torch.int32).contiguous(),
                kv_ptr=ptr(cols.sum(1)), kv_idx=cols.nonzero()[:, 1].to(torch.int32).contiguous())


def prepare(case, seed):
    c = case
    gen = torch.Generator(device="cuda").manual_seed(seed)
    s = dict(case=c, p=_problem(c), sel=_select(c))
    s["q"], s["k"] = _tokens(c, gen, c["hq"]), _tokens(c, gen, c["hkv"])
    if c["kind"] != "route":
        s["v"] = _tokens(c, gen, c["hkv"])
    if c["kind"] in ("op", "train", "coarse"):
        s["do"] = _tokens(c, gen, c["hq"], mean=False)
    if c["kind"] in ("op", "coarse"):
        s["gate"] = torch.randn((c["batch"], c["hq"], _cubes(c) * B), generator=gen, device="cuda")
    if c["kind"] == "coarse":
        s["of"] = torch.randn(s["q"].shape, generator=gen, device="cuda").to(_tdtype(c))
    if c["kind"] in ("forward", "train"):
        s.update(_lists(c, _mask(c, s["q"], s["k"])))
    if c["kind"] in ("path", "op", "route"):
        # the lists and scratch memory that such a program keeps between calls; -1
        # marks the entries past the live prefix (mass selection)
        p, sel = s["p"], s["sel"]
        cap = vsa2.vsa2_route_capacity(p, sel)[1]
        wsb = vsa2.vsa2_route_workspace(p, sel)[1]
        n = _cubes(c)

        def ints(m):
            return torch.full((m,), -1, dtype=torch.int32, device="cuda")

        s.update(cap=cap, wsb=wsb, ws=torch.empty(wsb, dtype=torch.uint8, device="cuda"),
                 row_ptr=ints(c["batch"] * c["hq"] * n + 1), col_idx=ints(cap),
                 kv_ptr=ints(c["batch"] * c["hkv"] * n + 1), kv_idx=ints(cap))
        if c["kind"] == "route":
            s["scores"] = torch.empty((c["batch"], c["hq"], n, n), dtype=torch.float32, device="cuda")
    return s


# --------------------------------------------------------------------------
# one pass
# --------------------------------------------------------------------------
def _route(s):
    c, p = s["case"], s["p"]
    r = (c["rt"], c["rh"], c["rw"])
    q_r, k_r = vsa2.pool(p, s["q"], r), vsa2.pool(p, s["k"], r)
    scores = s.get("scores")
    status = vsa2.vsa2_route(p, s["sel"], q_r.data_ptr(), k_r.data_ptr(), s["row_ptr"].data_ptr(),
                             s["col_idx"].data_ptr(), s["cap"], s["kv_ptr"].data_ptr(), s["kv_idx"].data_ptr(),
                             None if scores is None else scores.data_ptr(), s["ws"].data_ptr(), s["wsb"],
                             torch.cuda.current_stream().cuda_stream)
    if status:
        raise RuntimeError("vsa2_route: %s" % vsa2.STATUS_NAMES[status])
    return q_r, k_r


def _coarse_forward(s, o_f):
    p, full = s["p"], (4, 4, 4)
    qc, kc, vc = (vsa2.pool(p, s[x], full) for x in ("q", "k", "v"))
    o_c, lse_c = vsa2.coarse_fwd(p, qc, kc, vc)
    return (qc, kc, vc), o_c, lse_c, vsa2.gate_merge(p, s["gate"], o_c, o_f)


def _coarse_backward(s, means, o_c):
    p = s["p"]
    do_c, dgate = vsa2.gate_merge_bwd(p, s["gate"], o_c, s["do"])
    return do_c, dgate, vsa2.coarse_bwd(p, *means, do_c)


def run(state):
    s, p, kind = state, state["p"], state["case"]["kind"]
    if kind == "route":
        q_r, k_r = _route(s)
        return dict(q_r=q_r, k_r=k_r, scores=s["scores"], row_ptr=s["row_ptr"], col_idx=s["col_idx"],
                    kv_ptr=s["kv_ptr"], kv_idx=s["kv_idx"])
    if kind in ("path", "forward"):
        if kind == "path":
            _route(s)
        o, lse = vsa2.attn_fwd(p, s["q"], s["k"], s["v"], s["row_ptr"], s["col_idx"])
        return dict(o=o, lse=lse)
    if kind in ("train", "op"):
        # (o_lo, the rounding remainder of o, is handed on to the backward and
        # not compared: its bits depend on the last bit of o)
        if kind == "op":
            _route(s)
        o, lse, o_lo = vsa2.attn_fwd(p, s["q"], s["k"], s["v"], s["row_ptr"], s["col_idx"], training=True)
        out = dict(o=o, lse=lse)
        if kind == "op":
            means, o_c, lse_c, out["out"] = _coarse_forward(s, o)
            do_c, out["dgate"], grads_c = _coarse_backward(s, means, o_c)
        grads = vsa2.attn_bwd(p, s["q"], s["k"], s["v"], o, lse, s["do"], s["row_ptr"], s["col_idx"], s["kv_ptr"],
                              s["kv_idx"], o_lo=o_lo)
        if kind == "op":
            for g, g_c in zip(grads, grads_c):
                vsa2.unpool_add(p, g_c, g, (4, 4, 4))
        out.update(zip(("dq", "dk", "dv"), grads))
        return out
    means, o_c, lse_c, out = _coarse_forward(s, s["of"])
    do_c, dgate, grads_c = _coarse_backward(s, means, o_c)
    return dict(zip(("qc", "kc", "vc"), means), o_c=o_c, lse_c=lse_c, out=out, do_c=do_c, dgate=dgate,
                **dict(zip(("dq_c", "dk_c", "dv_c"), grads_c)))


# --------------------------------------------------------------------------
# what one pass cannot do without
# --------------------------------------------------------------------------
def work(case):
    c = case
    e, n, nb, d, g = _size(c), _cubes(c), _blocks(c), c["d"], _pooled(c)
    tq, tkv = c["batch"] * c["hq"] * nb * B, c["batch"] * c["hkv"] * nb * B       # tokens
    rq, rkv = c["batch"] * c["hq"] * n, c["batch"] * c["hkv"] * n                 # cube rows
    pairs = _pairs(c, _kept(c))
    byts, flops = 0, 0
    if c["kind"] in ("path", "op", "route"):
        byts += (tq + tkv) * d * e + 4 * (rq + rkv + 2 * rq * _kept(c))
        if c["kind"] == "route":
            byts += (rq + rkv) * g * d * e + 4 * rq * n
        flops += 2 * d * g * g * rq * n
    if c["kind"] in ("path", "op", "forward", "train"):
        byts += (tq + 2 * tkv) * d * e + tq * d * e + 4 * tq + 4 * pairs
        flops += 4 * B * B * d * pairs
    if c["kind"] in ("op", "train"):
        byts += 2 * tq * d * e + 2 * tkv * d * e        # dO read, dQ, dK, dV written
        flops += 10 * B * B * d * pairs
    if c["kind"] in ("op", "coarse"):
        byts += 2 * tq * d * e + 8 * tq                 # merged output, gate and its gradient
        flops += 14 * d * rq * n
    if c["kind"] == "coarse":
        byts += (2 * tq + 2 * tkv) * d * e + (4 * rq + 4 * rkv) * d * e
    return {"bytes": byts, "flops": flops}


# --------------------------------------------------------------------------
# tolerances
# --------------------------------------------------------------------------
def tolerance(case):
    """fp32: sums of the head dimension and of a row's keys in another order.
    bf16: P and dS enter the products rounded to 8 bits and the results are
    rounded again, 2^-9 relative each.  Selected indices follow the fp32 block
    scores; two scores closer than their rounding may swap, which shifts the
    indices between them in that row."""
    if case["kind"] == "route":
        return {"rel": 1e-5, "max": 1e-3, "differ": 2e-3}
    if case["dtype"] == "f32":
        return {"rel": 2e-5, "max": 2e-3}
    return {"rel": 1e-2, "max": 0.2}


# --------------------------------------------------------------------------
# 64-bit results
# --------------------------------------------------------------------------
def _pool64(c, x, r):
    """MeanPool of the video part over sub-cubes r, mean of the real tokens, rounded to the dtype."""
    n, g = _cubes(c), (4 // r[0], 4 // r[1], 4 // r[2])
    real = _real(c, x.device)[:n * B].double()

    def split(y, tail):
        y = y.reshape(*y.shape[:-2 if tail else -1], n, g[0], r[0], g[1], r[1], g[2], r[2], *([c["d"]] if tail else []))
        base = y.dim() - (7 if not tail else 8)
        return y.sum((base + 2, base + 4, base + 6))

    cnt = split(real, False).reshape(-1)                                # [n * G]
    heads = [split(x[b, h, :n * B].double() * real[:, None], True).reshape(-1, c["d"]) / cnt.clamp(min=1)[:, None]
             for b in range(x.shape[0]) for h in range(x.shape[1])]
    out = torch.stack(heads).reshape(x.shape[0], x.shape[1], -1, c["d"])
    return out.float().to(_tdtype(c)).double(), cnt > 0


def _scores64(c, q_r, k_r, live):
    """P_r [batch, hq, n, n]."""
    n, g, grp = _cubes(c), _pooled(c), c["hq"] // c["hkv"]
    weight = live.double().reshape(n, g)
    weight = weight / weight.sum(1, keepdim=True) / g                   # per pooled query of a cube
    out = torch.empty((c["batch"], c["hq"], n, n), dtype=torch.float64, device=q_r.device)
    step = max(1, min(n, int(2e8 // (n * g * g))))
    for b in range(c["batch"]):
        for h in range(c["hq"]):
            kt = k_r[b, h // grp].t().contiguous()
            for i in range(0, n, step):
                m = min(step, n - i)
                s = q_r[b, h, i * g:(i + m) * g] @ kt / math.sqrt(c["d"])
                s[:, ~live] = -math.inf
                p = torch.softmax(s, -1).reshape(m, g, n, g).sum(3)
                out[b, h, i:i + m] = (p * weight[i:i + m, :, None]).sum(1)
    return out


def _pick64(c, scores):
    """The rule's mask on 64-bit scores (top-k and mass)."""
    n = _cubes(c)
    p, idx = torch.sort(scores, dim=-1, descending=True, stable=True)
    rank = torch.arange(n, device=scores.device)
    if c["mode"] == MASS:
        take = (torch.cumsum(p, -1) - p < c["mass"] * p.sum(-1, keepdim=True)) & (rank < c["cap"])
    else:
        take = (rank < c["k"]).expand(p.shape)
    return torch.zeros(p.shape, dtype=torch.bool, device=p.device).scatter_(-1, idx, take)


def _attention64(c, q, k, v, do, mask):
    """o, lse and, with do, dq, dk, dv of the masked softmax attention."""
    nb, d, grp = _blocks(c), c["d"], c["hq"] // c["hkv"]
    real = _real(c, q.device)
    scale = 1 / math.sqrt(d)
    o, lse = torch.zeros(q.shape, dtype=torch.float64, device=q.device), torch.full(q.shape[:3], -math.inf,
                                                                                     dtype=torch.float64, device=q.device)
    dq = dk = dv = None
    if do is not None:
        dq = torch.zeros(q.shape, dtype=torch.float64, device=q.device)
        dk, dv = (torch.zeros(k.shape, dtype=torch.float64, device=q.device) for _ in range(2))
    counts = mask.sum(-1)
    for b in range(c["batch"]):
        for h in range(c["hq"]):
            hk = h // grp
            kb, vb = (x[b, hk].double().reshape(nb, B, d) for x in (k, v))
            # rows of one head in runs of about equal list length
            order = torch.argsort(counts[b, h], stable=True).tolist()
            longest = counts[b, h].tolist()
            i = 0
            while i < nb:
                top = longest[order[i]]
                j = i + 1
                while j < nb and longest[order[j]] <= max(1.3 * top, 4) and (j - i) * longest[order[j]] < 16000:
                    j += 1
                rows = torch.tensor(order[i:j], device=q.device)
                width = longest[order[j - 1]]
                i = j
                if width == 0:
                    continue
                sel = mask[b, h, rows]
                idx = torch.sort(sel.to(torch.int8), dim=-1, descending=True, stable=True)[1][:, :width]
                live = torch.gather(sel, 1, idx)
                ok = (live[:, :, None] & real.reshape(nb, B)[idx]).reshape(len(rows), 1, width * B)
                kg = kb[idx].reshape(len(rows), width * B, d)
                vg = vb[idx].reshape(len(rows), width * B, d)
                qb = q[b, h].reshape(nb, B, d)[rows].double()
                s = torch.bmm(qb, kg.transpose(1, 2).contiguous()).mul_(scale).masked_fill_(~ok, -math.inf)
                z = torch.logsumexp(s, -1)
                live_q = real.reshape(nb, B)[rows]
                p = torch.exp_(s.sub_(z[:, :, None])).mul_(live_q[:, :, None])
                ob = torch.bmm(p, vg)
                o[b, h].view(nb, B, d)[rows] = ob
                lse[b, h].view(nb, B)[rows] = torch.where(live_q, z, torch.full_like(z, -math.inf))
                if do is None:
                    continue
                g = do[b, h].reshape(nb, B, d)[rows].double()
                ds = torch.bmm(g, vg.transpose(1, 2).contiguous()).sub_((g * ob).sum(-1, keepdim=True)).mul_(p)
                dq[b, h].view(nb, B, d)[rows] = torch.bmm(ds, kg).mul_(scale)
                flat = idx.reshape(-1)
                for acc, w, x in ((dv, p, g), (dk, ds, qb * scale)):
                    acc[b, hk].view(nb, B, d).index_add_(
                        0, flat, torch.bmm(w.transpose(1, 2).contiguous(), x).reshape(-1, B, d))
    return o, lse, dq, dk, dv


def _coarse64(c, s, o_f):
    """The coarse branch in 64 bits: every output of the coarse case."""
    n, d, grp = _cubes(c), c["d"], c["hq"] // c["hkv"]
    qc, kc, vc = (_pool64(c, s[x], (4, 4, 4))[0] for x in ("q", "k", "v"))
    ke, ve = (x.repeat_interleave(grp, 1) for x in (kc, vc))
    real = _real(c, s["q"].device).double()
    shape = (c["batch"], c["hq"], n, B, d)
    th = torch.tanh(s["gate"].double())
    z = torch.matmul(qc, ke.transpose(2, 3).contiguous()) / math.sqrt(d)
    lse = torch.logsumexp(z, -1)
    p = torch.exp(z - lse[..., None])
    o_c = torch.matmul(p, ve)
    g = th.reshape(shape[:4]) * real.reshape(n, B)
    do_c, dgate = torch.empty_like(o_c), torch.empty_like(th)
    out = torch.empty(o_f.shape, dtype=torch.float64, device=o_f.device)
    for b in range(c["batch"]):
        for h in range(c["hq"]):
            do = s["do"][b, h].double().reshape(shape[2:])
            out[b, h] = (th[b, h].reshape(n, B, 1) * o_c[b, h][:, None] + o_f[b, h].reshape(n, B, d)).reshape(-1, d)
            do_c[b, h] = (g[b, h][..., None] * do).sum(1)
            dgate[b, h] = ((1 - th[b, h] ** 2) * (do * o_c[b, h][:, None]).sum(-1).reshape(-1)) * real
    dp = torch.matmul(do_c, ve.transpose(2, 3).contiguous())
    ds = p * (dp - (do_c * o_c).sum(-1, keepdim=True)) / math.sqrt(d)
    dq = torch.matmul(ds, ke)

    def fold(w, x):
        return torch.matmul(w.transpose(2, 3).contiguous(), x).reshape(c["batch"], c["hkv"], grp, n, d).sum(2)

    return dict(qc=qc, kc=kc, vc=vc, o_c=o_c, lse_c=lse, out=out, do_c=do_c, dgate=dgate, dq_c=dq,
                dk_c=fold(ds, qc), dv_c=fold(p, do_c))


def exact(case, seed):
    c = case
    kind, n = c["kind"], _cubes(c)
    fine = _pairs(c) if kind in ("path", "op", "forward", "train") else 0
    if fine * (1 if kind in ("path", "forward") else 3) > 6e6:
        return None                                     # over about 20 seconds
    s = prepare(c, seed)
    for x in ("ws", "col_idx", "kv_idx", "scores"):
        s.pop(x, None)
    if kind == "coarse":
        return _coarse64(c, s, s["of"].double())
    if kind in ("path", "op", "route"):
        r = (c["rt"], c["rh"], c["rw"])
        (q_r, live), (k_r, _) = _pool64(c, s["q"], r), _pool64(c, s["k"], r)
        scores = _scores64(c, q_r, k_r, live)
        if kind == "route":
            return dict(q_r=q_r, k_r=k_r, scores=scores, row_ptr=None, col_idx=None, kv_ptr=None, kv_idx=None)
        mask = _pick64(c, scores.float().double())
    else:
        mask = _mask(c, s["q"], s["k"])
    o, lse, dq, dk, dv = _attention64(c, s["q"], s["k"], s["v"], s.get("do"), mask)
    if kind in ("path", "forward"):
        return dict(o=o, lse=lse)
    out = dict(o=o, lse=lse, dq=dq, dk=dk, dv=dv)
    if kind == "op":
        grp = _coarse64(c, s, o)
        out.update(out=grp["out"], dgate=grp["dgate"])
        real = _real(c, dq.device).reshape(n, B)
        spread = real.double() / real.sum(1, keepdim=True)
        for name in ("dq", "dk", "dv"):
            g = out[name]
            for b in range(g.shape[0]):
                for h in range(g.shape[1]):
                    g[b, h].view(n, B, c["d"]).add_(spread[:, :, None] * grp[name + "_c"][b, h][:, None])
    return out
