"""The work that a user of the library has it do, as cases that can be timed and checked.

A case names an entry point, sizes, data type and options; `prepare` makes what a program holds
before the call, `run` is one pass through `paper_2608_20172_amd.binding`, and `exact` gives the
same outputs from plain torch in 64 bits (the definitions of `include/relation.h`, written out).

Kinds of case:
  relation  relation_fwd, or relation_fwd + relation_bwd (one training step of the operator)
  autograd  the same step through the differentiable wrapper `relation`
  layer     relation_layer_fwd + relation_layer_bwd: RoPE, Givens mixing and any head width
  decode    relation_decode: one new token per sequence against the KV cache
  linear    Linear Relation with the retention gate and RoPE: forward with the state (prefill),
            or forward + backward (a training step); "ungated" takes the log-retention itself
"""
from __future__ import annotations

import math

import torch

from paper_2608_20172_amd import binding as R

TAU = 2.0
ROPE_BASE = 1.0e4
DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}


def listed():
    return [
        # The smallest call: the fp32 parity workload's sizes, one training step. Launches and host time count.
        {"name": "step_tiny_fp32", "kind": "relation", "B": 1, "H": 2, "T": 128, "D": 32, "dtype": "f32", "step": True,
         "det": False, "layout": "bhtd", "std": 1.0, "boost": False},
        # Forward alone (evaluation, scoring) of a 10M-scale layer: few workgroups.
        {"name": "fwd_10m", "kind": "relation", "B": 8, "H": 4, "T": 512, "D": 64, "dtype": "bf16", "step": False,
         "det": False, "layout": "bhtd", "std": 0.125, "boost": False},
        # Training step of a 30M-scale layer through autograd, tensors as a model has them after
        # splitting a [B, T, H D] projection into heads.
        {"name": "autograd_30m", "kind": "autograd", "B": 8, "H": 8, "T": 1024, "D": 64, "dtype": "bf16",
         "layout": "bthd", "std": 0.125, "boost": False},
        # Training step of the 100M-scale layer, the benchmark's workload.
        {"name": "step_100m", "kind": "relation", "B": 8, "H": 12, "T": 2048, "D": 64, "dtype": "bf16", "step": True,
         "det": False, "layout": "bhtd", "std": 0.125, "boost": True},
        # Long context, the widest head: the largest case.
        {"name": "step_long", "kind": "relation", "B": 1, "H": 16, "T": 16384, "D": 128, "dtype": "bf16", "step": True,
         "det": False, "layout": "bhtd", "std": 1.0 / math.sqrt(128.0), "boost": False},
        # The paper's 100M model layer: 8 heads of width 80, RoPE and Givens mixing.
        {"name": "layer_100m", "kind": "layer", "B": 4, "H": 8, "T": 4096, "D": 80, "dtype": "bf16", "pairing": "A",
         "layout": "bthd", "std": 1.0},
        # The paper's 30M hybrid layer's width 60 (rows not on 16-byte boundaries), a ragged length, one micro-batch.
        {"name": "layer_ragged", "kind": "layer", "B": 4, "H": 8, "T": 1999, "D": 60, "dtype": "bf16", "pairing": "B",
         "layout": "bhtd", "std": 1.0},
        # Serving: a batch of sequences of mixed lengths.
        {"name": "decode_batch", "kind": "decode", "B": 64, "H": 12, "T": 4096, "D": 64, "dtype": "bf16", "low": 0.25,
         "std": 1.0},
        # Serving: one user with a long context.
        {"name": "decode_long", "kind": "decode", "B": 1, "H": 16, "T": 16384, "D": 128, "dtype": "bf16", "low": 1.0,
         "std": 1.0},
        # Linear Relation training step at its long context (the benchmark's largest at width 64).
        {"name": "linear_step_64", "kind": "linear", "B": 1, "H": 8, "T": 32768, "D": 64, "rope": 64, "dtype": "bf16",
         "step": True, "gate": "slow", "layout": "bhtd"},
        # The same layer at the 100M model's width 80 padded to 128, a micro-batch at its context.
        {"name": "linear_step_128", "kind": "linear", "B": 4, "H": 8, "T": 4096, "D": 128, "rope": 80, "dtype": "bf16",
         "step": True, "gate": "slow", "layout": "bhtd"},
        # Prefill of a prompt of odd length with the decode state, channels that forget fast among them.
        {"name": "linear_prefill", "kind": "linear", "B": 2, "H": 8, "T": 3001, "D": 64, "rope": 60, "dtype": "bf16",
         "step": False, "gate": "mixed", "layout": "bthd"},
    ]


# ---------------------------------------------------------------------------
# Drawn cases: the same kinds over their ranges
# ---------------------------------------------------------------------------
def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _length(rng, lo, hi):
    """A length over the logarithm of its range: half of them as they fall, half a multiple of 64."""
    t = int(round(_log(rng, lo, hi)))
    return max(lo, min(hi, (t + 63) // 64 * 64 if rng.random() < 0.5 else t))


def _heads(rng, T, budget, cap):
    """B and H (even) with B H at most what keeps B H T^2 within the budget."""
    most = max(2, min(cap, int(budget / (float(T) * T))))
    H = rng.choice([h for h in (2, 4, 8, 12, 16) if h <= most])
    B = max(1, min(most // H, int(round(_log(rng, 1, max(1.01, most / H))))))
    return B, H


def draw(rng):
    kind = rng.choice(["relation", "relation", "autograd", "layer", "layer", "decode", "decode", "linear", "linear"])
    dtype = "f32" if rng.random() < 0.15 else "bf16"
    layout = rng.choice(["bhtd", "bthd"])
    if kind in ("relation", "autograd", "layer"):
        D = rng.choice([32, 64, 64, 96, 128] if dtype == "bf16" else [32, 64, 128])
        if kind == "layer":
            D = rng.choice([48, 60, 64, 80])
        T = _length(rng, 64, 1024 if dtype == "f32" else 8192)
        B, H = _heads(rng, T, 1.5e9 if dtype == "bf16" else 1.0e8, 256)
        c = {"kind": kind, "B": B, "H": H, "T": T, "D": D, "dtype": dtype, "layout": layout}
        c["std"] = _log(rng, 1.0 / math.sqrt(D), 1.0)  # of q and k: evidence from near zero to unit variance
        if kind == "layer":
            c["pairing"] = rng.choice(["A", "B"])
            return c
        c["boost"] = rng.random() < 0.3
        if kind == "relation":
            c["step"] = rng.random() < 0.7
            c["det"] = c["step"] and rng.random() < 0.3
        return c
    if kind == "decode":
        D = rng.choice([64, 128]) if dtype == "f32" else rng.choice([64, 64, 96, 128])
        T = _length(rng, 128, 32768)
        H = rng.choice([4, 8, 12, 16])
        B = int(round(_log(rng, 1, max(1.01, min(128.0, 64 * 4096 / T)))))
        return {"kind": "decode", "B": B, "H": H, "T": T, "D": D, "dtype": dtype, "low": rng.uniform(0.1, 1.0), "std": 1.0}
    D = rng.choice([32, 64, 64, 128])
    T = _length(rng, 128, 32768)
    H = rng.choice([2, 4, 8])
    most = (32768 if dtype == "bf16" else 8192) * 8 // (2 if D == 128 else 1)
    T = min(T, most // H)
    B = int(round(_log(rng, 1, max(1.01, min(16.0, most / (T * H))))))
    gate = rng.choice(["slow", "mixed", "ungated"])
    rope = 0 if gate == "ungated" else rng.choice([0, D, {32: 24, 64: 60, 128: 80}[D]])
    return {"kind": "linear", "B": B, "H": H, "T": T, "D": D, "rope": rope, "dtype": dtype, "step": rng.random() < 0.6,
            "gate": gate, "layout": layout}


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------
def _gen(seed, dev):
    return torch.Generator(device=dev).manual_seed(int(seed))


def _tensor(c, g, std, dev):
    """[B, H, T, D] Gaussians in the case's type: contiguous, or a view of a [B, T, H, D] tensor."""
    B, H, T, D = c["B"], c["H"], c["T"], c["D"]
    shape = (B, T, H, D) if c["layout"] == "bthd" else (B, H, T, D)
    x = (torch.randn(shape, device=dev, generator=g) * std).to(DTYPES[c["dtype"]])
    return x.transpose(1, 2) if c["layout"] == "bthd" else x


def _lengths(c, g, dev):
    """Cache lengths spread evenly from low T to T, in an order of the seed (so their sum is the case's own)."""
    B, T = c["B"], c["T"]
    lens = torch.linspace(c["low"] * T, T, B, device=dev) if B > 1 else torch.full((1,), float(T), device=dev)
    lens = lens.round().clamp(1, T).to(torch.int32)
    return lens[torch.randperm(B, device=dev, generator=g)]


def prepare(c, seed):
    dev = torch.device("cuda:0")
    g = _gen(seed, dev)
    s = {"case": c}
    if c["kind"] == "decode":
        B, H, T, D = c["B"], c["H"], c["T"], c["D"]
        t = DTYPES[c["dtype"]]
        for name, std in (("k", c["std"]), ("v", 1.0)):
            s[name] = torch.randn(B, H, T, D, device=dev, generator=g).mul_(std).to(t)
        s["q"] = (torch.randn(B, H, D, device=dev, generator=g) * c["std"]).to(t)
        s["lengths"] = _lengths(c, g, dev)
        s["lam"] = torch.full((1,), 0.5, device=dev)  # the paper's initial value
        return s
    if c["kind"] == "linear":
        names = ["p1", "p2", "v"] + (["dout"] if c["step"] else [])
        for name in names:
            s[name] = _tensor(c, g, 1.0, dev)
        B, H, T, D = c["B"], c["H"], c["T"], c["D"]
        if c["gate"] == "ungated":  # log-retention -U(0, 0.05)
            s["r"] = torch.rand(B, H, T, D, device=dev, generator=g).mul_(-0.05)
            return s
        s["r"] = torch.randn(B, H, T, D, device=dev, generator=g)
        # "slow": retention of about 0.999 on every channel; "mixed": from 0.99 down to e^-5 a token
        am, ad, bm = (-4.0, 0.25, -3.0) if c["gate"] == "slow" else (0.0, 0.5, 0.0)
        s["a_log"] = am + ad * torch.randn(H, D, device=dev, generator=g)
        s["dt_bias"] = bm + torch.randn(H, D, device=dev, generator=g)
        return s
    for name in ("q", "k"):
        s[name] = _tensor(c, g, c["std"], dev)
    s["v"] = _tensor(c, g, c["std"], dev)
    if c.get("boost"):  # 5% of the query rows times 8
        rows = torch.rand(c["B"], c["H"], c["T"], 1, device=dev, generator=g) < 0.05
        s["q"].mul_(torch.where(rows, 8.0, 1.0).to(s["q"].dtype))
    if c.get("step", True):
        s["dout"] = _tensor(c, g, 1.0, dev)
    s["lam"] = torch.full((1,), 0.5, device=dev)
    if c["kind"] == "layer":
        s["theta"] = (torch.rand(c["H"] // 2, device=dev, generator=g) * 2 - 1) * math.pi
    if c["kind"] == "autograd":
        for name in ("q", "k", "v", "lam"):
            s[name].requires_grad_(True)
    return s


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------
def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "relation":
        f = R.relation_fwd(s["q"], s["k"], s["v"], s["lam"])
        out = {"o": f["o"], "row_stat": f["row_stat"]}
        if c["step"]:
            g = R.relation_bwd(s["q"], s["k"], s["v"], f["o"], s["dout"], s["lam"], f["row_stat"],
                               deterministic=c["det"])
            out.update({n: g[n] for n in ("dq", "dk", "dv", "dlambda")})
        return out
    if kind == "autograd":
        o = R.relation(s["q"], s["k"], s["v"], s["lam"])
        dq, dk, dv, dlam = torch.autograd.grad(o, (s["q"], s["k"], s["v"], s["lam"]), s["dout"])
        return {"o": o.detach(), "dq": dq, "dk": dk, "dv": dv, "dlambda": dlam}
    if kind == "layer":
        f = R.relation_layer_fwd(s["q"], s["k"], s["v"], s["lam"], s["theta"], pairing=c["pairing"])
        g = R.relation_layer_bwd(s["q"], s["k"], s["v"], f["o"], s["dout"], s["lam"], f["row_stat"], s["theta"],
                                 saved=f["saved"], pairing=c["pairing"])
        return {"o": f["o"], "row_stat": f["row_stat"], **{n: g[n] for n in ("dq", "dk", "dv", "dlambda", "dtheta")}}
    if kind == "decode":
        return R.relation_decode(s["q"], s["k"], s["v"], s["lengths"], s["lam"])
    if c["gate"] == "ungated":
        f = R.relation_linear_fwd(s["p1"], s["p2"], s["v"], s["r"], want_state=not c["step"])
        if not c["step"]:
            return f
        return {"o": f["o"], **R.relation_linear_bwd(s["p1"], s["p2"], s["v"], s["r"], s["dout"])}
    f = R.relation_linear_gated_fwd(s["p1"], s["p2"], s["v"], s["r"], s["a_log"], s["dt_bias"], rope_dim=c["rope"],
                                    want_state=not c["step"])
    if not c["step"]:
        return f
    return {"o": f["o"], **R.relation_linear_gated_bwd(s["p1"], s["p2"], s["v"], s["r"], s["a_log"], s["dt_bias"],
                                                       s["dout"], rope_dim=c["rope"])}


# ---------------------------------------------------------------------------
# The work that a pass cannot do without
# ---------------------------------------------------------------------------
def work(c):
    B, H, T, D = c["B"], c["H"], c["T"], c["D"]
    es = 2 if c["dtype"] == "bf16" else 4
    x = B * H * T * D
    if c["kind"] == "decode":
        keys = sum(T if B == 1 else min(T, max(1, round(c["low"] * T + i * (1 - c["low"]) * T / (B - 1)))) for i in range(B))
        # K and V rows of every valid entry; q in, o and row_stat out
        return {"bytes": H * keys * D * 2 * es + 2 * B * H * D * es + 4 * B * H, "flops": 4.0 * H * keys * D}
    if c["kind"] == "linear":
        if c["step"]:  # p1, p2, v, dY, r in; y, dp1, dp2, dv, dr out; three times the forward's products
            return {"bytes": 8 * es * x + 8 * x, "flops": 12.0 * x * D}
        # p1, p2, v, r in; y and the state out; one read and one update of a D x D state per token
        return {"bytes": 4 * es * x + 4 * x + 4 * B * H * D * D, "flops": 4.0 * x * D}
    pairs = B * H * T * (T - 1) / 2
    if c.get("step", True):  # q, k, v, dO in; o, row statistic, dq, dk, dv out
        return {"bytes": 8 * es * x + 4 * B * H * T, "flops": 14.0 * D * pairs}
    return {"bytes": 4 * es * x + 4 * B * H * T, "flops": 4.0 * D * pairs}


def tolerance(c):
    # 2-norms against `exact`, measured: 32-bit cases 4e-7 at most; bf16 operator, decode and Linear Relation
    # 2.4e-3 (outputs rounded to bf16, products of bf16 operands); layers 5e-3 (their prepared operands are
    # rounded to bf16 too). The signed sums dlambda and dtheta cancel, hence the wider bar of the passes that return them.
    if c["dtype"] == "f32":
        return {"rel": 1.0e-5}
    signed_sums = c["kind"] in ("autograd", "layer") or c["kind"] == "relation" and c["step"]
    return {"rel": 2.0e-2 if signed_sums else 1.0e-2}


# ---------------------------------------------------------------------------
# The same outputs in 64 bits
# ---------------------------------------------------------------------------
def _relation64(q, k, v, lam, scale, dout=None):
    """Causal Full Relation of one head ([T, D] fp64) in blocks of rows: y, M and, with dout, dq, dk, dv, dlambda."""
    T = q.shape[0]
    o, M = torch.empty_like(v), torch.empty(T, dtype=q.dtype, device=q.device)
    dq, dk, dv = torch.zeros_like(q), torch.zeros_like(k), torch.zeros_like(v)
    dlam = torch.zeros((), dtype=q.dtype, device=q.device)
    for a in range(0, T, 2048):
        b = min(T, a + 2048)
        i = torch.arange(a, b, device=q.device)
        j = torch.arange(b, device=q.device)
        ln = torch.log((i + 1).to(q.dtype))
        U = scale * (q[a:b] @ k[:b].t())
        sg = torch.sigmoid(U)
        own = j[None] == i[:, None]
        S = torch.sigmoid(U / TAU)
        E = U * sg
        Rm = torch.where(own, S, E - lam * ln[:, None]).masked_fill(j[None] > i[:, None], -math.inf)
        lse = torch.logsumexp(Rm, 1)
        F = torch.exp(Rm - lse[:, None])
        o[a:b] = F @ v[:b]
        M[a:b] = lse + lam * ln
        if dout is None:
            continue
        G = dout[a:b]
        dR = F * (G @ v[:b].t() - (G * o[a:b]).sum(1)[:, None])
        dU = dR * torch.where(own, S * (1 - S) / TAU, sg + E * (1 - sg))
        dq[a:b] = scale * (dU @ k[:b])
        dk[:b] += scale * (dU.t() @ q[a:b])
        dv[:b] += F.t() @ G
        dlam -= (ln * dR.masked_fill(own, 0.0).sum(1)).sum()
    return o, M, dq, dk, dv, dlam


def _relation64_all(q, k, v, lam, scale, dout=None):
    B, H = q.shape[:2]
    per = [_relation64(q[b, h], k[b, h], v[b, h], lam, scale, None if dout is None else dout[b, h])
           for b in range(B) for h in range(H)]
    back = [torch.stack([p[n] for p in per]).unflatten(0, (B, H)) for n in range(5)]
    return back + [sum(p[5] for p in per).reshape(1)]


def _rope64(x, rope_dim, base=ROPE_BASE):
    """Channel j of the first rope_dim with channel j + rope_dim / 2 by t base^(-2 j / rope_dim)."""
    if rope_dim == 0:
        return x
    h = rope_dim // 2
    t = torch.arange(x.shape[2], dtype=x.dtype, device=x.device)
    ang = t[:, None] * base ** (-2.0 * torch.arange(h, dtype=x.dtype, device=x.device) / rope_dim)
    cs, sn = torch.cos(ang), torch.sin(ang)
    a, b = x[..., :h], x[..., h:rope_dim]
    return torch.cat([a * cs - b * sn, a * sn + b * cs, x[..., rope_dim:]], -1)


def _givens64(v, theta, pairing):
    """Head pairs (1, 2), (3, 4), ... of pairing A or (2, 3), ..., (H, 1) of B, turned by theta."""
    H = v.shape[1]
    first = torch.arange(0, H, 2, device=v.device) + (0 if pairing == "A" else 1)
    second = (first + 1) % H
    cs, sn = torch.cos(theta)[None, :, None, None], torch.sin(theta)[None, :, None, None]
    a, b = v[:, first], v[:, second]
    order = torch.argsort(torch.cat([first, second]))
    return torch.cat([cs * a - sn * b, sn * a + cs * b], 1)[:, order]


def _linear64(p1, p2, v, g, scale, rope_dim, L=16):
    """Linear Relation over [N, T, D] fp64 in chunks of L tokens (every exponent <= 0): y and the last state."""
    N, T, D = v.shape
    S = torch.sigmoid(scale * (p1 * p2).sum(-1, keepdim=True) / TAU)
    q, k = (_rope64((S * p / p.norm(dim=-1, keepdim=True))[None], rope_dim)[0] for p in (p1, p2))
    pad = -T % L
    q, k, vv, g = (torch.nn.functional.pad(x, (0, 0, 0, pad)).reshape(N, -1, L, D) for x in (q, k, v, g))
    b = g.cumsum(2)
    below = torch.ones(L, L, dtype=torch.bool, device=v.device).tril(-1)[:, :, None]
    A = []
    for c in range(0, q.shape[1], 256):  # pairs inside a chunk, some chunks at a time
        s = slice(c, c + 256)
        w = torch.exp((b[:, s, :, None] - b[:, s, None]).masked_fill(~below, -math.inf))
        A.append((q[:, s, :, None] * k[:, s, None] * w).sum(-1))
    y = vv + torch.cat(A, 1) @ vv
    last = b[:, :, -1:]
    add = (k * torch.exp(last - b)).transpose(2, 3).contiguous() @ vv
    keep = torch.exp(last[:, :, 0])[..., None]
    C, before = torch.zeros_like(add[:, 0]), []
    for kc, ac in zip(keep.unbind(1), add.unbind(1)):
        before.append(C)
        C = kc * C + ac
    y = y + (q * torch.exp(b)) @ torch.stack(before, 1)
    return y.reshape(N, -1, D)[:, :T], C


def exact(c, seed):
    s = prepare(c, seed)
    x = {n: t.detach().double() for n, t in s.items() if torch.is_tensor(t) and t.is_floating_point()}
    B, H, T, D = c["B"], c["H"], c["T"], c["D"]
    scale = 1.0 / math.sqrt(D)
    if c["kind"] == "decode":
        o, M = torch.empty(B, H, D, dtype=torch.float64, device=x["q"].device), torch.empty(B, H, dtype=torch.float64, device=x["q"].device)
        for b, n in enumerate(s["lengths"].tolist()):
            U = scale * (x["k"][b, :, :n] @ x["q"][b, :, :, None])[..., 0]
            Rm = U * torch.sigmoid(U) - x["lam"] * math.log(n)
            Rm[:, -1] = torch.sigmoid(U[:, -1] / TAU)
            lse = torch.logsumexp(Rm, 1)
            o[b] = (torch.exp(Rm - lse[:, None])[:, None] @ x["v"][b, :, :n])[:, 0]
            M[b] = lse + x["lam"] * math.log(n)
        return {"o": o, "row_stat": M}
    if c["kind"] == "linear":
        names = ["p1", "p2", "v", "r"] + ([] if c["gate"] == "ungated" else ["a_log", "dt_bias"])
        leaf = {n: x[n].clone().requires_grad_(c["step"]) for n in names}
        g = leaf["r"]
        if c["gate"] != "ungated":
            g = -torch.exp(leaf["a_log"])[None, :, None] * torch.nn.functional.softplus(g + leaf["dt_bias"][None, :, None], threshold=700)
        with torch.set_grad_enabled(c["step"]):
            y, C = _linear64(*(t.reshape(B * H, T, D) for t in (leaf["p1"], leaf["p2"], leaf["v"], g)), scale, c["rope"])
            y = y.reshape(B, H, T, D)
        if not c["step"]:
            return {"o": y, "state": C.reshape(B, H, D, D)}
        grads = torch.autograd.grad(y, [leaf[n] for n in names], x["dout"])
        called = {"r": "dg" if c["gate"] == "ungated" else "dr", "a_log": "da_log", "dt_bias": "ddt_bias"}
        return {"o": y.detach(), **{called.get(n, "d" + n): t for n, t in zip(names, grads)}}
    lam = x["lam"][0]
    if c["kind"] == "layer":
        leaf = [x[n].clone().requires_grad_(True) for n in ("q", "k", "v", "theta")]
        mixed = [_rope64(leaf[0], D), _rope64(leaf[1], D), _givens64(leaf[2], leaf[3], c["pairing"])]
        o, M, dq, dk, dv, dlam = _relation64_all(*(t.detach() for t in mixed), lam, scale, x["dout"])
        dq, dk, dv, dth = torch.autograd.grad(mixed, leaf, [dq, dk, dv])
        return {"o": o, "row_stat": M, "dq": dq, "dk": dk, "dv": dv, "dlambda": dlam, "dtheta": dth}
    o, M, dq, dk, dv, dlam = _relation64_all(x["q"], x["k"], x["v"], lam, scale, x.get("dout"))
    if c["kind"] == "autograd":
        return {"o": o, "dq": dq, "dk": dk, "dv": dv, "dlambda": dlam}
    out = {"o": o, "row_stat": M}
    if c["step"]:
        out.update({"dq": dq, "dk": dk, "dv": dv, "dlambda": dlam})
    return out
