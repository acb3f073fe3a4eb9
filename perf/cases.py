"""Workloads of the LaCT fast-weight layer through its public entry points.

Each case is one call (or one short chain of calls) that a program makes of
this package: the layer's forward over a sequence as a model serves it, the
backward as it trains it, the linear fast weight, and the streaming steps on
either side of the path. Shapes are the language-model, novel-view-synthesis
and video workloads of ``lact_synth.CONFIGS``, shortened where Muon makes the
chunk recurrence chaotic (a perturbation grows about twofold per chunk, so a
long run cannot be compared), plus ragged lengths.

``op``: "forward", "backward" (SwiGLU or, with ``linear``, the linear fast
weight), "train" (forward, then backward) or "layer_io" (prologue, output
RMSNorm and their reverses).
"""
from __future__ import annotations

import math

import torch

import paper_2505_23884_amd as P

A, B, C = 3.4445, -4.7750, 2.0315   # Newton-Schulz quintic (App. A, Details of Muon)
EPS = 1e-7
NS_STEPS = 5
LR_BIAS = -4.6


def _case(name, op, b, heads, d, h, n_kv, n_q, chunk, order=0, muon=False, momentum=False, lr3=False, linear=False,
          fp32=False, schedule=False):
    c = {"op": op, "B": b, "H": heads, "d": d, "h": h, "n_kv": n_kv, "n_q": n_q, "chunk": chunk, "order": order,
         "muon": muon, "momentum": momentum, "lr3": lr3, "linear": linear, "fp32": fp32, "schedule": schedule}
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: a small fp32 layer, four short chunks (launches and latency)
        _case("tiny_fp32", "forward", 1, 2, 64, 64, 1024, 1024, 256, fp32=True),
        # one prompt of a served language model, ragged last chunk, momentum optimizer
        _case("lm_prompt", "forward", 1, 4, 512, 512, 5003, 5003, 1024, momentum=True),
        # the language-model prefill that the benchmark times: a batch of 32K-token sequences
        _case("lm32k", "forward", 4, 4, 512, 512, 32768, 32768, 2048),
        # the full language-model optimizer (Muon, momentum, a rate per matrix), two chunks
        _case("lm_muon_mom", "forward", 4, 4, 512, 512, 4096, 4096, 2048, muon=True, momentum=True, lr3=True),
        # novel-view synthesis: one 256K-token chunk of input views, then the target views
        _case("nvs256k", "forward", 1, 1, 768, 1536, 262144, 266240, 262144, order=1),
        # video: many narrow heads, Muon, frame chunks of 3120 tokens, the last one partial
        _case("video", "forward", 1, 40, 128, 256, 9001, 9001, 3120, muon=True),
        # teacher-forced video diffusion: noisy chunks apply only, clean ones update then apply
        _case("video_tf", "forward", 1, 40, 128, 256, 15600, 15600, 3120, muon=True, schedule=True),
        # training: the reverse of the language-model sequence
        _case("lm32k_bwd", "backward", 4, 4, 512, 512, 32768, 32768, 2048),
        # training with the full language-model optimizer
        _case("lm_muon_mom_bwd", "backward", 4, 4, 512, 512, 4096, 4096, 2048, muon=True, momentum=True, lr3=True),
        # training on video
        _case("video_bwd", "backward", 1, 40, 128, 256, 6240, 6240, 3120, muon=True),
        # a training step of the linear fast weight, ragged last chunk
        _case("linear_train", "train", 4, 4, 512, 512, 16001, 16001, 2048, linear=True),
        # the layer's steps on either side of the path in a training step
        _case("layer_io", "layer_io", 2, 4, 512, 512, 32768, 32768, 2048, momentum=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        op = rng.choice(["forward", "forward", "forward", "backward", "backward", "train", "layer_io"])
        if op == "layer_io":
            n = _log_int(rng, 500, 40000)
            return _case(None, op, rng.randint(1, 3), rng.randint(1, 8), 32 * rng.randint(2, 24), 512, n, n, 2048,
                         momentum=rng.random() < 0.5, lr3=rng.random() < 0.5, fp32=rng.random() < 0.2)
        linear = op == "train" or rng.random() < 0.1
        muon = not linear and rng.random() < 0.4
        fp32 = rng.random() < 0.15
        d = 32 * rng.randint(2, 24)
        h = d if linear else 32 * rng.randint(2, 32) if rng.random() < 0.5 else d * rng.choice([1, 2])
        bh = rng.choice([(1, rng.randint(1, 4)), (rng.randint(1, 4), 4), (1, rng.randint(8, 40))])
        if muon:   # at most two whole-rank updates (one in the backward, whose reverse is the worse
            # conditioned), a last chunk of most of the chunk's length
            chunk = max(_log_int(rng, 1024, 4096), 4 * max(d, h))
            n = chunk * (rng.randint(1, 2) if op == "forward" else 1) - rng.randint(0, chunk // 4)
        else:
            chunk = _log_int(rng, 256, 16384)
            n = _log_int(rng, 700, 131072)
        order = rng.randint(0, 1)
        schedule = op == "forward" and not linear and rng.random() < 0.15
        tail = 0 if schedule or (rng.random() < 0.6 and not (muon and op == "backward")) else rng.randint(1, 2000)
        if schedule:
            n += n if n % 2 else n + 1
        c = _case(None, op, *bh, d, h, n, n + tail, chunk, order, muon, rng.random() < 0.4,
                  not linear and rng.random() < 0.3, linear, fp32, schedule)
        w = work(c)
        if w["flops"] <= (1e11 if fp32 else 2.5e12) and w["bytes"] <= 3e9 and n / chunk <= 64:
            return c


def _segments(c):
    """Teacher forcing: noisy and clean stretches of `chunk` tokens in turn."""
    n, ch = c["n_kv"], c["chunk"]
    return [("apply_only" if i % 2 == 0 else "update_then_apply", t, min(n, t + ch))
            for i, t in enumerate(range(0, n, ch))]


def _io(c):
    return torch.float32 if c["fp32"] else torch.bfloat16


def prepare(case, seed):
    c = case
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev).manual_seed(int(seed))
    nb, nh, d, h = c["B"], c["H"], c["d"], c["h"]
    io = _io(c)

    def randn(*shape):
        return torch.randn(*shape, generator=gen, device=dev)

    s = {"case": c}
    if c["op"] == "layer_io":
        n = c["n_q"]
        s["qkv"] = randn(nb, n, 3, nh, d).to(io)
        s["lr_raw"] = randn(nb, n, nh, *((3,) if c["lr3"] else ()))
        s["beta_raw"] = randn(nb, n, nh) if c["momentum"] else None
        s["o"], s["norm_w"] = randn(nb, nh, n, d).to(io), 1.0 + 0.1 * randn(nh, d)
        s["dy"] = randn(nb, n, nh, d).to(io)
        s["dq"], s["dk"], s["dv"] = (randn(nb, nh, n, d).to(io) for _ in range(3))
        s["deta"] = randn(nb, nh, n, *((3,) if c["lr3"] else ()))
        s["dbeta"] = randn(nb, nh, n) if c["momentum"] else None
        return s

    def tokens(n):
        x = randn(nb, nh, n, d)
        return (x / x.norm(dim=-1, keepdim=True)).to(io)

    def weight(r, k):
        w = randn(nh, r, k)
        w = w / w.norm(dim=-1, keepdim=True)
        return w.unsqueeze(0).expand(nb, nh, r, k).contiguous()

    s["q"], s["k"], s["v"] = tokens(c["n_q"]), tokens(c["n_kv"]), tokens(c["n_kv"])
    s["eta"] = 0.01 * torch.nn.functional.softplus(randn(nb, nh, c["n_kv"], *((3,) if c["lr3"] else ())))
    s["beta"] = torch.sigmoid(randn(nb, nh, c["n_kv"])) if c["momentum"] else None
    shapes = [(d, d)] if c["linear"] else [(h, d), (d, h), (h, d)]
    s["W"] = [weight(*x) for x in shapes]
    if c["op"] != "forward":
        s["dout"] = (randn(nb, nh, c["n_q"], d) / math.sqrt(d)).to(io)
        s["M"] = [1e-3 / math.sqrt(d) * randn(nb, nh, *x) for x in shapes] if c["momentum"] else None
    return s


def _forward(s):
    """The layer's forward from its initial fast weights (kept: the entry points update them in place)."""
    c = s["case"]
    W = [w.clone() for w in s["W"]]
    M = [m.clone() for m in s["M"]] if s.get("M") else None
    q, k, v, eta, muon = s["q"], s["k"], s["v"], s["eta"], c["muon"]
    if c["schedule"]:
        r = P.forward_schedule(q, k, v, eta, *W, _segments(c), use_muon=muon, beta=s["beta"])
    elif c["linear"]:
        r = P.forward_linear(q, k, v, eta, W[0], c["chunk"], c["order"], use_muon=muon, beta=s["beta"],
                             M=M[0] if M else None)
    elif c["momentum"]:
        r = P.forward_momentum(q, k, v, eta, s["beta"], *W, *(M or ()), chunk=c["chunk"], order=c["order"],
                               use_muon=muon)
    else:
        r = P.forward(q, k, v, eta, *W, chunk=c["chunk"], order=c["order"], use_muon=muon)
    return [r, W]


def _backward(s):
    c = s["case"]
    q, k, v, eta, W, dout, muon = s["q"], s["k"], s["v"], s["eta"], s["W"], s["dout"], c["muon"]
    if c["momentum"]:
        one = c["linear"]
        return P.backward_momentum(q, k, v, eta, s["beta"], W[0] if one else W, s["M"][0] if one else s["M"], dout,
                                   c["chunk"], c["order"], use_muon=muon)
    if c["linear"]:
        return P.backward_linear(q, k, v, eta, W[0], dout, c["chunk"], c["order"], use_muon=muon)
    return P.backward(q, k, v, eta, *W, dout, c["chunk"], c["order"], use_muon=muon)


def run(state):
    s = state
    op = s["case"]["op"]
    if op == "layer_io":
        fwd = P.prologue(s["qkv"], s["lr_raw"], LR_BIAS, s["beta_raw"])
        y = P.rmsnorm_out(s["o"], s["norm_w"])
        dn = P.rmsnorm_out_backward(s["o"], s["dy"], s["norm_w"])
        dp = P.prologue_backward(s["qkv"], s["lr_raw"], LR_BIAS, s["beta_raw"], s["dq"], s["dk"], s["dv"], s["deta"],
                                 s["dbeta"])
        return [fwd, y, dn, dp]
    if op == "forward":
        return _forward(s)
    if op == "backward":
        return _backward(s)
    return [_forward(s), _backward(s)]


def _updates(c):
    """Lengths of the update steps and the number of applied tokens."""
    if c["schedule"]:
        segs = _segments(c)
        return [e - b for m, b, e in segs if m != "apply_only"], c["n_q"]
    return [min(c["chunk"], c["n_kv"] - t) for t in range(0, c["n_kv"], c["chunk"])], c["n_q"]


def work(case):
    """Each input read once and each output written once; the contractions of the method (the
    backward's count has the replayed update: its entry points are given the initial weights)."""
    c = case
    bh, d, h = c["B"] * c["H"], c["d"], c["h"]
    e = 4 if c["fp32"] else 2
    if c["op"] == "layer_io":
        n = c["n_q"]
        rates = (3 if c["lr3"] else 1) + (1 if c["momentum"] else 0)
        vec = 3 + 3 + 1 + 1 + 2 + 1 + 3 + 3 + 3   # prologue, norm, and their reverses
        return {"bytes": bh * n * (vec * d * e + 5 * rates * 4.0), "flops": bh * n * d * 60.0}
    ups, nq = _updates(c)
    nk = sum(ups)
    mats = [(d, d)] if c["linear"] else [(h, d), (d, h), (h, d)]
    state = bh * sum(r * k for r, k in mats) * 4.0 * (2 if c["momentum"] else 1)
    lo, hi = min(d, h), max(d, h)
    ns = len(mats) * NS_STEPS * (4.0 * lo * lo * hi + 2.0 * lo ** 3) * len(ups) if c["muon"] else 0.0
    rates = (3 if c["lr3"] else 1) + (1 if c["momentum"] else 0)
    ins = bh * ((nq + 2 * nk) * d * e + nk * rates * 4.0) + state
    out = bh * nq * d * e
    flops = nbytes = 0.0
    if c["op"] in ("forward", "train"):
        flops += bh * ((2.0 * d * d * (nk + nq)) if c["linear"] else (12.0 * nk + 6.0 * nq) * d * h) + bh * ns
        nbytes += ins + out + state
    if c["op"] in ("backward", "train"):
        flops += bh * ((6.0 * nk + 4.0 * nq) * d * d if c["linear"] else (36.0 * nk + 16.0 * nq) * d * h)
        flops += bh * 3.0 * ns
        nbytes += 2 * ins + out
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """About four times what the path shows against `exact` (bf16 operands and
    intermediates; fp16 Newton-Schulz operands with Muon; fp32 throughout)."""
    c = case
    if c["op"] == "layer_io":
        return {"rel": 2e-6, "max": 1e-4} if c["fp32"] else {"rel": 8e-3, "max": 2e-2}
    if c["fp32"]:
        return {"rel": 4e-4 if c["muon"] else 1e-5}
    if c["muon"]:
        return {"rel": 3e-2}
    return {"rel": 1.6e-2}


# ---- the same in 64 bits, plain torch --------------------------------------

def _silu(z):
    return z * torch.sigmoid(z)


def _apply(W, x):
    if len(W) == 1:
        return x @ W[0].T
    return (_silu(x @ W[0].T) * (x @ W[2].T)) @ W[1].T


def _neg_gradient(W, k, v, eta):
    """-g of the chunk's loss: sum over tokens of eta f_W(k)^T v differentiated in W."""
    if len(W) == 1:
        return [(eta[:, :1] * v).T @ k]
    out = None
    r1, r2, r3 = (eta[:, j:j + 1] for j in range(3)) if eta.shape[1] == 3 else (eta,) * 3
    z1, z3, c = k @ W[0].T, k @ W[2].T, v @ W[1]
    sg = torch.sigmoid(z1)
    a = z1 * sg
    out = [(r1 * c * z3 * (sg + a * (1 - sg))).T @ k, (r2 * v).T @ (a * z3), (r3 * c * a).T @ k]
    return out


def _newton_schulz(g):
    tall = g.shape[0] > g.shape[1]
    x = g.T if tall else g
    x = x / (x.norm() + EPS)
    for _ in range(NS_STEPS):
        m = x @ x.T
        x = A * x + (B * m + C * (m @ m)) @ x
    return x.T if tall else x


def _update(W, M, k, v, eta, beta, muon, block=32768):
    if torch.is_grad_enabled() or k.shape[0] <= block:
        p = _neg_gradient(W, k, v, eta)
    else:
        p = [torch.zeros_like(w) for w in W]
        for t in range(0, k.shape[0], block):
            part = _neg_gradient(W, k[t:t + block].double(), v[t:t + block].double(), eta[t:t + block])
            p = [x + y for x, y in zip(p, part)]
    if M is not None:
        bb = beta.mean()
        M = [bb * m - x for m, x in zip(M, p)]
        p = [-m for m in M]
    if muon:
        p = [_newton_schulz(x) for x in p]
    new = []
    for w, x in zip(W, p):
        u = w + x
        new.append(u * (w.norm(dim=1, keepdim=True) / u.norm(dim=1, keepdim=True)))
    return new, M


def _instance(c, q, k, v, eta, beta, W, M):
    """One (batch, head): outputs, final weights and final momentum."""
    segs = _segments(c) if c["schedule"] else [
        ("apply_then_update" if c["order"] == 0 else "update_then_apply", t, min(c["n_kv"], t + c["chunk"]))
        for t in range(0, c["n_kv"], c["chunk"])]
    if not c["schedule"] and c["n_q"] > c["n_kv"]:
        segs.append(("apply_only", c["n_kv"], c["n_q"]))
    o = []
    for mode, b, e in segs:
        if mode in ("apply_only", "apply_then_update"):
            o.append(_apply(W, q[b:e]))
        if mode != "apply_only":
            W, M = _update(W, M, k[b:e], v[b:e], eta[b:e], None if beta is None else beta[b:e], c["muon"])
        if mode == "update_then_apply":
            o.append(_apply(W, q[b:e]))
    return torch.cat(o), W, M


def _flat(t, trailing):
    """[B, H, ...] -> [B*H, ...] in 64 bits, `trailing` axes kept."""
    return t.reshape(-1, *t.shape[-trailing:]).double()


def _exact_path(c, s):
    bh, d = c["B"] * c["H"], c["d"]
    W0 = [_flat(w, 2) for w in s["W"]]
    M0 = [_flat(m, 2) for m in s["M"]] if s.get("M") else None
    if M0 is None and c["momentum"]:
        M0 = [torch.zeros_like(w) for w in W0]
    eta = s["eta"].reshape(bh, c["n_kv"], -1)
    beta = s["beta"].reshape(bh, -1) if c["momentum"] else None
    flat = {x: s[x].reshape(bh, -1, d) for x in ("q", "k", "v")}
    want_f, want_b = c["op"] != "backward", c["op"] != "forward"
    outs, Ws, Ms, grads = [], [], [], []
    for i in range(bh):
        ins = [flat[x][i].double() for x in ("q", "k", "v")] + [eta[i].double()]
        if c["momentum"]:
            ins.append(beta[i].double())
        ins += [w[i].clone() for w in W0] + ([m[i].clone() for m in M0] if M0 else [])
        if want_b:
            ins = [x.requires_grad_() for x in ins]
        nw, at = len(W0), 5 if c["momentum"] else 4
        with torch.set_grad_enabled(want_b):
            o, W, M = _instance(c, *ins[:4], ins[4] if c["momentum"] else None, ins[at:at + nw],
                                ins[at + nw:] if M0 else None)
        if want_f:
            outs.append(o.detach())
            Ws.append([w.detach() for w in W])
            Ms.append([m.detach() for m in M] if M0 else None)
        if want_b:
            g = torch.autograd.grad(o, ins, s["dout"].reshape(bh, -1, d)[i].double(), allow_unused=True)
            grads.append([torch.zeros_like(x) if y is None else y for x, y in zip(ins, g)])
        del o, W, M, ins

    def stack(xs, like):
        return torch.stack(xs).reshape(like.shape)

    res = []
    if want_f:
        o = stack(outs, s["q"])
        Wl = [stack([x[j] for x in Ws], w) for j, w in enumerate(s["W"])]
        if M0:
            Ml = [stack([x[j] for x in Ms], w) for j, w in enumerate(s["W"])]
            res.append([(o, Ml[0] if c["linear"] else tuple(Ml)), Wl])
        else:
            res.append([o, Wl])
    if want_b:
        like = [s["q"], s["k"], s["v"], s["eta"]] + ([s["beta"]] if c["momentum"] else []) + s["W"] + (s["M"] or [])
        g = [stack([x[j] for x in grads], t) for j, t in enumerate(like)]
        if c["momentum"]:
            nw = len(s["W"])
            dW, dM = g[5:5 + nw], g[5 + nw:]
            g = (*g[:5], dW[0], dM[0]) if c["linear"] else (*g[:5], tuple(dW), tuple(dM))
        res.append(tuple(g))
    return res if c["op"] == "train" else res[0]


def _exact_io(c, s):
    heads = lambda t: t.transpose(1, 2)   # [B, L, H, ..] <-> [B, H, L, ..]
    ins = [s[x].double().requires_grad_() for x in ("qkv", "lr_raw")]
    if c["momentum"]:
        ins.append(s["beta_raw"].double().requires_grad_())
    u = _silu(ins[0])
    q, k = (heads(u[:, :, j] / u[:, :, j].norm(dim=-1, keepdim=True)) for j in range(2))
    v = heads(u[:, :, 2])
    eta = heads(torch.nn.functional.softplus(ins[1] + LR_BIAS))
    outs = [q, k, v, eta] + ([heads(torch.sigmoid(ins[2]))] if c["momentum"] else [])
    cot = [s[x].double() for x in ("dq", "dk", "dv", "deta")] + ([s["dbeta"].double()] if c["momentum"] else [])
    g = torch.autograd.grad(outs, ins, cot)
    fwd = tuple(x.detach() for x in outs) + (() if c["momentum"] else (None,))
    dp = tuple(g) + (() if c["momentum"] else (None,))
    del outs, u
    o, w = s["o"].double().requires_grad_(), s["norm_w"].double().requires_grad_()
    y = heads(o * torch.rsqrt((o * o).mean(dim=-1, keepdim=True) + 1e-6) * w[:, None, :])
    dn = torch.autograd.grad(y, [o, w], s["dy"].double())
    return [fwd, y.detach(), tuple(dn), dp]


def exact(case, seed):
    c = case
    s = prepare(c, seed)
    return _exact_io(c, s) if c["op"] == "layer_io" else _exact_path(c, s)
