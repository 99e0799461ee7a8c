"""Timing cases of the LinSimp library: the calls a user's program makes, through
the public binding (paper_2608_09307_amd.linsimp), over the supported range.

The cases stand for five uses: inference forwards, training steps (forward and
backward on one shared workspace), the full head's training step, prefill of a
decode state, and autoregressive decode (one token, or a few at a time).

A case is a dict of plain values:
  op     "fwd"     forward; scratch "static" (fwd_static) or "own" (caller workspace)
         "train"   forward + backward, the backward reusing the forward's states
         "head"    head forward + backward (L2 norm, core, gated RMSNorm)
         "prefill" decode state from a prefix
         "decode"  one token for every sequence
         "chunk"   T consecutive tokens for every sequence in one call
  B (sequences), H (heads), n (tokens), D (= Dv), m (features), w (window),
  dtype "bf16" or "f32", and per op: scratch, gate, boost, T.
"""

from __future__ import annotations

import ctypes
import math

import torch

from paper_2608_09307_amd import linsimp as L
from paper_2608_09307_amd.workloads import Workload, make_head_params, make_inputs

LOG2E = 1.4426950408889634
DEV = "cuda"

# (D, m) with a bf16 or float32 kernel
BF16_SHAPES = ((32, 32), (64, 64), (64, 128), (128, 64), (128, 128), (128, 256))
F32_SHAPES = ((32, 32), (32, 64), (64, 32), (64, 64))


def listed():
    return [
        # one small head in a tight serving loop: latency and launches
        dict(name="fwd_head_f32_n256", op="fwd", scratch="static", B=1, H=1, n=256, D=32, m=32, w=64, dtype="f32"),
        # inference forward (scoring) of the 2k-token layer
        dict(name="fwd_layer2k", op="fwd", scratch="own", B=4, H=8, n=2048, D=64, m=64, w=64, dtype="bf16"),
        # training step of the layer the paper times
        dict(name="train_layer2k_m128", op="train", B=8, H=6, n=2048, D=64, m=128, w=64, dtype="bf16", boost=1.0),
        # training step of the 16k-token layer (the throughput workload)
        dict(name="train_layer16k", op="train", B=2, H=16, n=16384, D=128, m=128, w=64, dtype="bf16", boost=1.0),
        # training step of the long-context layer with two feature blocks and large keys
        dict(name="train_stress64k_m256", op="train", B=1, H=32, n=65536, D=128, m=256, w=64, dtype="bf16", boost=4.0),
        # training step of the full head: wide window, ragged length, channel-wise gate
        dict(name="train_head_n3001_w100", op="head", B=2, H=8, n=3001, D=128, m=64, w=100, dtype="bf16", gate="channel"),
        # float32 training step (gradient checks, small models), ragged length and window
        dict(name="train_f32_n1000_w48", op="train", B=2, H=4, n=1000, D=64, m=64, w=48, dtype="f32", boost=1.0),
        # one long prompt: time to first token of an interactive session
        dict(name="prefill_prompt16k", op="prefill", B=1, H=16, n=16384, D=128, m=128, w=64, dtype="bf16"),
        # a batch of prompts
        dict(name="prefill_64x8k", op="prefill", B=64, H=16, n=8192, D=128, m=128, w=64, dtype="bf16"),
        # one interactive stream: a token at a time
        dict(name="decode_1seq", op="decode", B=1, H=16, n=1, D=128, m=128, w=64, dtype="bf16"),
        # batched serving: a token for every sequence
        dict(name="decode_256seq", op="decode", B=256, H=16, n=1, D=128, m=128, w=64, dtype="bf16"),
        # several tokens a call (draft verification, short continuations)
        dict(name="chunk_32seq_t16", op="chunk", B=32, H=16, n=1, D=128, m=128, w=64, dtype="bf16", T=16),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(("fwd", "train", "train", "head", "prefill", "decode", "chunk"))
    dtype = "f32" if rng.random() < 0.2 else "bf16"
    D, m = rng.choice(F32_SHAPES if dtype == "f32" else BF16_SHAPES)
    # the paper's windows (64, 32), any width up to 64, and wider ones where m allows
    pick = rng.random()
    w = 64 if pick < 0.4 else 32 if pick < 0.5 else rng.randint(1, 64)
    if m <= 64 and not (dtype == "f32" and D == 64 and m == 64) and rng.random() < 0.15:
        w = rng.randint(65, 128)
    H = rng.choice((1, 2, 4, 6, 8, 12, 16, 32))
    c = dict(op=op, B=1, H=H, n=1, D=D, m=m, w=w, dtype=dtype)
    if op in ("decode", "chunk"):
        c["B"] = _log_int(rng, 1, 256)
        if op == "chunk":
            c["T"] = _log_int(rng, 2, 64)
            c["B"] = min(c["B"], 64)
        return c
    c["n"] = _log_int(rng, 100, 32768)
    c["B"] = _log_int(rng, 1, 16)
    while c["B"] * H * c["n"] > 1 << 19 and c["B"] > 1:
        c["B"] -= 1
    if op == "fwd":
        c["scratch"] = "own"
    elif op == "train":
        c["boost"] = rng.choice((1.0, 1.0, 4.0))
    elif op == "head":
        c["gate"] = rng.choice(("head", "channel"))
    return c


def _workload(c, seed):
    boost = c.get("boost", 1.0)
    return Workload("case", c["B"], c["H"], c["n"], c["D"], c["D"], c["m"], c["w"], c["dtype"],
                    "fwdbwd" if c["op"] in ("train", "head") else "fwd",
                    boost_frac=0.05 if boost != 1.0 else 0.0, boost=boost, seed=seed)


def _layer_tensors(c, seed):
    x = make_inputs(_workload(c, seed), device=DEV)
    boosted = x.pop("boost_mask", None)
    if boosted is not None:
        # a sequence opens with an ordinary key
        x["k"][:, :, 0] /= torch.where(boosted[:, None, :1], c["boost"], 1.0).to(x["k"].dtype)
    return x


def _decode_tensors(c, seed):
    """State after a prefix (built here from 256 random tokens), every sequence at
    a length of its own, and T new tokens."""
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    dt = torch.float32 if c["dtype"] == "f32" else torch.bfloat16
    S, H, D, m, w, P = c["B"], c["H"], c["D"], c["m"], c["w"], 256
    s = D ** -0.25

    def stream(*shape):
        return (torch.randn(shape, generator=g, device=DEV) * s).to(dt)

    omega = torch.randn((H, m, D), generator=g, device=DEV)
    M = torch.empty(S, H, m, D, device=DEV)
    a = torch.empty(S, H, m, device=DEV)
    rho = torch.empty(S, H, device=DEV)
    for s0 in range(0, S, 32):
        s1 = min(S, s0 + 32)
        k = stream(s1 - s0, H, P, D).float()
        v = stream(s1 - s0, H, P, D).float()
        lam = (k @ omega.transpose(1, 2).contiguous() - 0.5 * k.square().sum(-1, keepdim=True)) * LOG2E
        top = lam.amax((2, 3))
        chi = torch.exp2(lam - top[..., None, None]) / math.sqrt(m)
        M[s0:s1] = chi.transpose(2, 3).contiguous() @ v
        a[s0:s1] = chi.sum(2)
        rho[s0:s1] = top
    state = {"M": M, "a": a, "rho": rho, "ring_r": stream(S, H, w, D), "ring_u": stream(S, H, w, D),
             "pos": torch.randint(P, 8192, (S,), generator=g, device=DEV, dtype=torch.int64)}
    tok = (c["T"],) if c["op"] == "chunk" else ()
    x = {name: stream(S, H, *tok, D) for name in "qkvru"}
    return state, x, omega


def _prefill_tensors(c, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    dt = torch.float32 if c["dtype"] == "f32" else torch.bfloat16
    shape = (c["B"], c["H"], c["n"], c["D"])
    x = {}
    for name in "kvru":
        t = torch.empty(shape, dtype=dt, device=DEV)
        for b in range(c["B"]):
            t[b] = torch.randn(shape[1:], generator=g, device=DEV) * c["D"] ** -0.25
        x[name] = t
    return x, torch.randn((c["H"], c["m"], c["D"]), generator=g, device=DEV)


def prepare(case, seed):
    c, op = case, case["op"]
    st = {"case": c}
    if op in ("decode", "chunk"):
        st["state"], st["x"], st["omega"] = _decode_tensors(c, seed)
        return st
    if op == "prefill":
        st["x"], st["omega"] = _prefill_tensors(c, seed)
        x = st["x"]
        d = L.make_dims(c["B"], c["H"], c["n"], c["D"], c["D"], c["m"], c["w"], L._dtype_code(x["k"]))
        st["workspace"] = L.alloc_workspace(d, False, x["k"].device)
        return st
    wl = _workload(c, seed)
    x = st["x"] = _layer_tensors(c, seed)
    d = L.dims_of(x["q"], x["v"], x["omega"], c["w"])
    if op == "head":
        # raw streams: the head normalises q, k, r itself
        st.update(make_head_params(wl, device=DEV, channel_gate=c["gate"] == "channel"))
        st["workspace"] = L._aligned_bytes(int(L.lib().linsimp_head_workspace_size(ctypes.byref(d), 1)), x["q"].device)
    elif op == "train":
        st["workspace"] = L.alloc_workspace(d, True, x["q"].device)
    elif c["scratch"] == "own":
        st["workspace"] = L.alloc_workspace(d, False, x["q"].device)
    return st


def run(state):
    c, op, w = state["case"], state["case"]["op"], state["case"]["w"]
    if op in ("decode", "chunk"):
        x, s = state["x"], state["state"]
        step = L.decode_step if op == "decode" else L.decode_chunk
        out = step(s, x["q"], x["k"], x["v"], x["r"], x["u"], state["omega"], w)
        return {"out": out, **s}
    if op == "prefill":
        x = state["x"]
        return L.prefill(x["k"], x["v"], x["r"], x["u"], state["omega"], w, workspace=state["workspace"])
    x = state["x"]
    args = (x["q"], x["k"], x["v"], x["r"], x["u"], x["omega"], w)
    if op == "fwd":
        if c["scratch"] == "static":
            return L.fwd_static(*args, want_stats=False)[0]
        return L.fwd(*args, workspace=state["workspace"], want_stats=False)[0]
    if op == "train":
        out, stats = L.fwd(*args, workspace=state["workspace"])
        grads = L.bwd(*args, out, stats, x["dO"], workspace=state["workspace"], reuse_states=True)
        return [out, *grads]
    y, saved = L.head_fwd(*args, state["tau"], state["gate"], workspace=state["workspace"])
    grads = L.head_bwd(*args, state["tau"], state["gate"], saved, x["dO"], workspace=state["workspace"],
                       reuse_states=True)
    return [y, *grads]


def work(case):
    """Each input read once, each output written once; the method's own
    contractions (2 operations a multiply-add)."""
    c = case
    e = 2 if c["dtype"] == "bf16" else 4
    B, H, n, D, m, w, op = c["B"], c["H"], c["n"], c["D"], c["m"], c["w"], c["op"]
    bank = H * m * D * 4
    pair, tok = 2 * m * (2 * D + 1), 2 * m * (2 * D + 1)
    if op in ("decode", "chunk"):
        T = c.get("T", 1)
        state = 2 * 4 * (m * (D + 1) + 1) + e * 2 * D * (w + min(T, w))
        return {"bytes": B * H * (state + e * 6 * D * T) + bank, "flops": B * H * T * (tok + w * pair)}
    rows = B * H * n
    if op == "prefill":
        ring = min(n, w) + w
        return {"bytes": e * 2 * D * rows + B * H * (4 * (m * (D + 1) + 1) + e * 2 * D * ring) + bank,
                "flops": rows * tok}
    pairs = B * H * (n * (n + 1) // 2 if n <= w else w * (w + 1) // 2 + (n - w) * w)
    flops = pairs * pair + rows * tok
    if op == "fwd":
        return {"bytes": e * 6 * D * rows + bank, "flops": flops}
    # backward: five contractions a pair, four a token; inputs again, dO, five gradients
    flops += pairs * 2 * m * 5 * D + rows * 2 * m * 4 * D
    streams = 5 + 1 + 1 + 5 + (2 if op == "head" and c["gate"] == "channel" else 0)
    return {"bytes": e * streams * D * rows + bank, "flops": flops}


def tolerance(case):
    """About four times the largest error of an output against 64 bits seen over
    the ranges: forward and decode outputs 3.6e-3 (bf16), prefilled states
    1.5e-3, gradients 5.9e-3; float32 1.5e-6.  "max": single elements of long
    gradients cancel between the much larger values of the rows around them."""
    if case["dtype"] == "f32":
        return {"rel": 6e-6, "max": 2.4e-4}
    if case["op"] == "prefill":
        return {"rel": 6e-3, "max": 0.2}
    if case["op"] in ("train", "head"):
        return {"rel": 2.4e-2, "max": 0.99}
    return {"rel": 1.5e-2, "max": 0.6}


# ---------------------------------------------------------------------------
# 64-bit values in plain torch
# ---------------------------------------------------------------------------

def _exact_sequence(q, k, v, r, u, om, w, dO):
    """One (sequence, head): out and, with dO, (dq, dk, dv, dr, du); float64.
    Blocks of 64 rows, each against the state before it and its own tokens."""
    C = 64
    n, D = k.shape
    nb = -(-n // C)
    pad = nb * C - n
    one = torch.ones(n, 1, dtype=torch.float64, device=k.device)
    lam = k @ om.t().contiguous() - 0.5 * k.square().sum(-1, keepdim=True)
    chi = torch.exp(lam - lam.max())

    def rows(x):
        return torch.cat([x, x.new_zeros(pad, x.shape[1])]).view(nb, C, -1)

    chib, ve, qb = rows(chi), rows(torch.cat([v, one], 1)), rows(q)
    cont = chib.transpose(1, 2).contiguous() @ ve
    # exclusive sums by a shift: their terms differ by many orders of magnitude
    Mb = torch.zeros_like(cont)
    Mb[1:] = cont[:-1].cumsum(0)
    idx = torch.arange(nb, device=k.device)[:, None] * C + torch.arange(C + w - 1, device=k.device)[None] - (w - 1)
    inside = (idx >= 0) & (idx < n)
    at = idx.clamp(0, n - 1)
    ue = torch.cat([u, one], 1)
    causal = torch.tril(torch.ones(C, C, dtype=torch.float64, device=k.device))[None, :, None, :]
    grad = dO is not None
    out = torch.empty(nb, C, D, dtype=torch.float64, device=k.device)
    if grad:
        dOb = rows(dO)
        dq, dchi, dve, dM = (torch.zeros_like(t) for t in (qb, chib, ve, Mb))
        dr, du = torch.zeros(n, D, dtype=torch.float64, device=k.device), torch.zeros_like(ue)
    G = max(1, (1 << 29) // (C * w * om.shape[0] * 8 * (2 if grad else 1)))
    for g0 in range(0, nb, G):
        s = slice(g0, min(nb, g0 + G))
        ok = inside[s]
        leaf = [t.detach().clone().requires_grad_(grad) for t in
                (qb[s], r[at[s]] * ok[..., None], ue[at[s]] * ok[..., None], chib[s], ve[s], Mb[s])]
        lq, lr, lu, lc, lv, lM = leaf
        z = lq[:, :, None, :] * lr.unfold(1, w, 1).transpose(2, 3)                 # [G, C, w, D]
        ell = z @ om.t().contiguous() - 0.5 * z.square().sum(-1, keepdim=True)
        # anchors before the sequence; rows past its end keep theirs (their outputs are dropped)
        ell = ell.masked_fill(~(idx[s] >= 0).unfold(1, w, 1)[..., None], -math.inf)
        psi = torch.exp(ell - ell.detach().amax((2, 3), keepdim=True))
        g = psi.shape[0]
        flat = psi.reshape(g, C * w, -1)
        P = (flat @ lc.transpose(1, 2).contiguous()).view(g, C, w, C) * causal
        A = flat @ lM + P.reshape(g, C * w, C) @ lv
        NZ = (A.view(g, C, w, -1) * lu.unfold(1, w, 1).transpose(2, 3)).sum(2)
        o = NZ[..., :D] / (NZ[..., D:] + 1e-300)
        out[s] = o.detach()
        if grad:
            gq, gr, gu, gc, gv, gM = torch.autograd.grad((o * dOb[s]).sum(), leaf)
            dq[s], dchi[s], dve[s], dM[s] = gq, gc, gv, gM
            dr.index_add_(0, at[s].reshape(-1), (gr * ok[..., None]).reshape(-1, D))
            du.index_add_(0, at[s].reshape(-1), (gu * ok[..., None]).reshape(-1, D + 1))
    out = out.view(nb * C, D)[:n]
    if not grad:
        return out, None
    dcont = torch.zeros_like(dM)                             # gradient of each block's contribution
    dcont[:-1] = dM[1:].flip(0).cumsum(0).flip(0)
    dchi = (dchi + ve @ dcont.transpose(1, 2).contiguous()).view(nb * C, -1)[:n]
    dve = (dve + chib @ dcont).view(nb * C, -1)[:n]
    dlam = dchi * chi
    dk = dlam @ om - dlam.sum(-1, keepdim=True) * k
    return out, (dq.view(nb * C, D)[:n], dk, dve[:, :D], dr, du[:, :D])


def _exact_core(q, k, v, r, u, omega, w, dO=None):
    B, H = q.shape[:2]
    out, grads = torch.empty_like(v), [torch.empty_like(t) for t in (q, k, v, r, u)] if dO is not None else None
    for b in range(B):
        for h in range(H):
            o, gs = _exact_sequence(q[b, h], k[b, h], v[b, h], r[b, h], u[b, h], omega[h], w,
                                    None if dO is None else dO[b, h])
            out[b, h] = o
            for t, g in zip(grads or (), gs or ()):
                t[b, h] = g
    return out, grads


def _exact_decode(c, seed):
    state, x, omega = _decode_tensors(c, seed)
    om = omega.double()
    omT = om.transpose(1, 2).contiguous()
    st = {k: (v.clone() if k == "pos" else v.double()) for k, v in state.items()}
    x = {k: v.double() for k, v in x.items()}
    S, H, w, m = c["B"], c["H"], c["w"], c["m"]
    T = c.get("T", 1)
    if c["op"] == "decode":
        x = {k: v.unsqueeze(2) for k, v in x.items()}
    si = torch.arange(S, device=DEV)
    outs = []
    for j in range(T):
        q, k, v, r, u = (x[n][:, :, j] for n in "qkvru")
        lam = ((k[:, :, None, :] @ omT).squeeze(2) - 0.5 * k.square().sum(-1, keepdim=True)) * LOG2E
        new = torch.maximum(st["rho"], lam.amax(-1))
        scale = torch.exp2(st["rho"] - new)[..., None]
        chi = torch.exp2(lam - new[..., None]) / math.sqrt(m)
        st["M"] = st["M"] * scale[..., None] + chi[..., None] * v[:, :, None, :]
        st["a"] = st["a"] * scale + chi
        st["rho"] = new
        slot = st["pos"] % w
        st["ring_r"][si, :, slot] = r
        st["ring_u"][si, :, slot] = u
        st["pos"] += 1                                       # (every sequence is past its first window)
        z = q[:, :, None, :] * st["ring_r"]
        ell = z @ omT - 0.5 * z.square().sum(-1, keepdim=True)
        psi = torch.exp(ell - ell.amax((2, 3), keepdim=True))
        N = ((psi @ st["M"]) * st["ring_u"]).sum(2)
        Z = (psi * st["a"][:, :, None, :]).sum((2, 3))
        outs.append(N / Z[..., None])
    out = outs[0] if c["op"] == "decode" else torch.stack(outs, 2)
    return {"out": out, **{k: None if k == "pos" else v for k, v in st.items()}}


def _exact_prefill(c, seed):
    x, omega = _prefill_tensors(c, seed)
    S, H, n, w, m, D = c["B"], c["H"], c["n"], c["w"], c["m"], c["D"]
    M = torch.empty(S, H, m, D, dtype=torch.float64, device=DEV)
    a = torch.empty(S, H, m, dtype=torch.float64, device=DEV)
    rho = torch.empty(S, H, dtype=torch.float64, device=DEV)
    for s in range(S):
        for h in range(H):
            k, v, om = x["k"][s, h].double(), x["v"][s, h].double(), omega[h].double()
            lam = (k @ om.t().contiguous() - 0.5 * k.square().sum(-1, keepdim=True)) * LOG2E
            rho[s, h] = lam.max()
            chi = torch.exp2(lam - rho[s, h]) / math.sqrt(m)
            M[s, h], a[s, h] = chi.t().contiguous() @ v, chi.sum(0)
    ring = {}
    for name in "ru":
        t = torch.zeros(S, H, w, D, dtype=torch.float64, device=DEV)
        j = torch.arange(max(0, n - w), n, device=DEV)
        t[:, :, j % w] = x[name][:, :, j].double()
        ring["ring_" + name] = t
    return {"M": M, "a": a, "rho": rho, **ring, "pos": None}


def exact(case, seed):
    c, op = case, case["op"]
    if op in ("decode", "chunk"):
        return _exact_decode(c, seed)
    if op == "prefill":
        return _exact_prefill(c, seed)
    wl = _workload(c, seed)
    raw = _layer_tensors(c, seed)
    x = {k: t.double() for k, t in raw.items()}
    if op == "fwd":
        return _exact_core(x["q"], x["k"], x["v"], x["r"], x["u"], x["omega"], c["w"])[0]
    if op == "train":
        out, grads = _exact_core(x["q"], x["k"], x["v"], x["r"], x["u"], x["omega"], c["w"], x["dO"])
        return [out, *grads]
    p = make_head_params(wl, device=DEV, channel_gate=c["gate"] == "channel")
    q, k, r, tau, gate = (t.double().requires_grad_() for t in (raw["q"], raw["k"], raw["r"], p["tau"], p["gate"]))
    norm = torch.nn.functional.normalize
    qn, kn, rn = norm(q, dim=-1) * tau[:, None, None], norm(k, dim=-1), norm(r, dim=-1)
    core = (qn.detach(), kn.detach(), x["v"], rn.detach(), x["u"], x["omega"], c["w"])
    o = _exact_core(*core)[0].requires_grad_()
    g = torch.sigmoid(gate if gate.dim() == 4 else gate[:, None, None])
    y = g * o / torch.sqrt(o.square().mean(-1, keepdim=True) + 1e-6)
    do, dgate = torch.autograd.grad((y * x["dO"]).sum(), [o, gate])
    dqn, dkn, dv, drn, du = _exact_core(*core, do)[1]
    dq, dk, dr, dtau = torch.autograd.grad([qn, kn, rn], [q, k, r, tau], [dqn, dkn, drn])
    return [y.detach(), dq, dk, dv, dr, du, dtau, dgate]
