"""The work that programs have this library do, as measurable cases.

A case is one call of one public entry point (``forward``, ``backward``, ``step``, ``decay_forward``,
``decay_step``, ``layer_forward``) at one size.  ``listed()`` gives the standing cases, ``draw`` one
more of the same ranges, ``prepare`` what a program has in hand before the call, ``run`` the call,
and ``exact`` the same outputs in float64 by plain torch.
"""
from __future__ import annotations

import math

import torch

import paper_2606_09862_amd as bla

DEV = "cuda:0"
F64 = torch.float64


def listed():
    return [
        # Serving one conversation: one token through one layer, the tables kept from the first step.
        # The smallest call: latency and launches count.
        _case("decode_one", "step", B=1, H=16, M=64, S=64, t0=2048),
        # Serving a full batch, every row at its own position (continuous batching): the state
        # traffic of 8192 heads.
        _case("decode_batch", "step", B=512, H=16, M=64, S=64, t0=2048, rows=True),
        # Decoding with the state-decay form at the paper's slot count 2M-1.
        _case("decay_decode", "decay_step", B=64, H=16, M=64, S=127, t0=1000, rows=True),
        # Prefill of one prompt of an odd length: few sequences, so their tokens have to fill the chip.
        # A plain call: no kept workspace, tables built by the call.
        _case("prompt", "forward", B=1, H=16, L=2000, M=64, S=64, keep=False),
        # Recall task (MQAR shape) with the paper's efficient form: anchored slots, S = 2M-1.
        _case("recall_anchored", "forward", B=64, H=4, L=512, M=32, S=63, anchor=True),
        # One layer of a language model in training or batch prefill: the benchmark workload.
        _case("lm_forward", "forward", B=8, H=16, L=4096, M=64, S=64),
        # Long documents with wide heads and many modes: the largest call.
        _case("long_context", "forward", B=1, H=16, L=65536, d=128, M=128, S=128),
        # Full-precision evaluation of a small model, continued from an earlier state at an odd
        # length, the paper's slot count.
        _case("f32_continue", "forward", dtype="f32", B=8, H=4, L=1000, M=32, S=63, t0=511, state=True, keep=False),
        # Training step of the language-model layer: gradients of q, k, v and of the input states.
        _case("lm_backward", "backward", B=8, H=16, L=4096, M=64, S=64),
        # Training step of the recall task at the paper's slot count, a ragged length and a carried
        # state (truncated backpropagation).
        _case("recall_backward", "backward", B=64, H=4, L=500, M=32, S=63, t0=500, state=True),
        # The state-decay form over the language-model layer's tokens.
        _case("decay_forward", "decay_forward", B=8, H=16, L=4096, M=64, S=64),
        # A whole layer of the recall model: projections, operator, output projection.
        _case("layer", "layer", B=64, H=4, L=512, M=32, S=32),
    ]


def _case(name, kind, *, B, H, M, S, L=1, d=64, dtype="bf16", t0=0, anchor=False, state=False, keep=True,
          rows=False):
    """keep: the program keeps the workspace (and, where the entry point can, the tables in it);
    state: the call continues from an input state; rows: each row of a decode step has its own position."""
    c = dict(kind=kind, dtype=dtype, B=B, H=H, L=L, d=d, M=M, S=S, t0=t0, anchor=anchor, state=state,
             keep=keep, rows=rows)
    if name:
        c["name"] = name
    return c


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.499)))))))


# Most operations (work()["flops"]) of a drawn case per kind: within the cost of the largest listed one.
_DRAW_FLOPS = {"forward": 2.5e10, "f32": 2.0e9, "backward": 5.0e10, "decay_forward": 1.2e10, "layer": 2.0e10}


def draw(rng):
    kind = rng.choice(["forward", "forward", "forward", "backward", "backward", "step", "decay_forward",
                       "decay_step", "layer"])
    dtype = "f32" if kind in ("forward", "step", "decay_step") and rng.random() < 0.3 else "bf16"
    while True:
        if kind == "backward":
            d, M = rng.choice([32, 64, 64]), _log_int(rng, 8, 64)
        elif kind == "forward" and dtype == "bf16":
            d, M = rng.choice([32, 64, 64, 128]), _log_int(rng, 8, 128)
        elif kind == "layer":
            d, M = rng.choice([32, 64, 64, 128]), _log_int(rng, 8, 64)
        else:
            d, M = rng.choice([32, 64, 64]), _log_int(rng, 8, 64)
        S = rng.choice([M, 2 * M - 1, 2 * M - 1])
        H = rng.choice([1, 2, 4, 6, 8, 12, 16])
        step = kind in ("step", "decay_step")
        B = _log_int(rng, 1, 512) if step else _log_int(rng, 1, 64)
        L = 1 if step else _log_int(rng, 64, 16384)
        state = rng.random() < 0.4 and kind != "layer"
        t0 = rng.randrange(0, 4096) if (step or state) else 0
        c = _case(None, kind, dtype=dtype, B=B, H=H, L=L, d=d, M=M, S=S, t0=t0, state=state,
                  anchor=kind in ("forward", "step") and rng.random() < 0.4, keep=rng.random() < 0.6,
                  rows=step and rng.random() < 0.5)
        cap = _DRAW_FLOPS.get("f32" if dtype == "f32" else kind, 1e30)
        if work(c)["flops"] <= cap and B * H * L <= 1 << 20:
            return c


def work(case):
    B, H, L, d, M, S = (case[x] for x in ("B", "H", "L", "d", "M", "S"))
    e = 4 if case["dtype"] == "f32" else 2
    th = B * H * L                      # token-heads
    modes = 2 * B * H * 2 * M * d * 4   # key and value mode states, float32
    slots = 2 * B * H * S * d * 4
    kind = case["kind"]
    states = 1 + int(case["state"])     # final states written, input states read
    if kind in ("forward", "layer"):
        # state update 8Md, query against the state 4Md, readout 4Md, slot scores and weights 4MS each
        flops = th * (16 * M * d + 8 * M * S)
        if kind == "forward":
            return {"bytes": th * 4 * d * e + states * modes, "flops": flops}
        D = H * d
        return {"bytes": 2 * B * L * D * e + 4 * D * D * e + modes, "flops": flops + B * L * 8 * D * D}
    if kind == "backward":
        # forward state, its query and output-gradient products, dq, dk, dv and the adjoint update; four
        # products with the slot matrices
        return {"bytes": th * 7 * d * e + states * modes, "flops": th * (36 * M * d + 16 * M * S)}
    if kind == "step":
        return {"bytes": th * 4 * d * e + 2 * modes, "flops": th * (24 * M * d + 8 * M * S)}
    if kind == "decay_step":
        return {"bytes": th * 4 * d * e + 2 * slots, "flops": th * 10 * S * d}
    return {"bytes": th * 4 * d * e + states * slots, "flops": th * 10 * S * d}


def tolerance(case):
    # Some four times the largest difference from float64 that was measured over the listed and some
    # drawn cases.
    if case["dtype"] == "f32":
        return {"rel": 4e-6}    # 8.1e-7: float32 products and sums over up to a thousand tokens
    if case["kind"] == "backward":
        return {"rel": 2.5e-2}  # 5.8e-3: products of bf16-rounded scores, weights and states, twice over
    if case["kind"] == "layer":
        return {"rel": 2e-2}    # 4.7e-3: bf16 between the projections and the operator
    return {"rel": 2e-2}        # 6.6e-3: bf16 operands and tables, float32 sums


# ------------------------------------------------------------------------------------- inputs

def _periods(case):
    """Heads alternate between token resolution 1 and 2: T = (1 + h mod 2)(2M-1)."""
    return [float((1 + h % 2) * (2 * case["M"] - 1)) for h in range(case["H"])]


def _dtype(case):
    return torch.float32 if case["dtype"] == "f32" else torch.bfloat16


def _inputs(case, seed):
    """Queries ~ N(0,1)/sqrt(d), keys and values ~ N(0,1) (projections of normalised hidden states);
    states as some hundreds of such tokens leave them."""
    g = torch.Generator(device=DEV)
    g.manual_seed(1000003 * seed + 17)
    B, H, L, d, M, S = (case[x] for x in ("B", "H", "L", "d", "M", "S"))
    dt, kind = _dtype(case), case["kind"]

    def normal(*shape, scale=1.0, dtype=dt):
        return torch.randn(*shape, generator=g, device=DEV, dtype=torch.float32).mul_(scale).to(dtype)

    x = {}
    if kind == "layer":
        D = H * d
        x["x"] = normal(B, L, D)
        x["w_qkv"] = normal(D, 3 * D, scale=D ** -0.5)
        x["w_qkv"][:, :D].mul_(0.25)  # queries at the scale of a trained model's: soft, not one-hot, weights
        x["w_o"] = normal(D, D, scale=D ** -0.5)
        return x
    shape = (B, H, d) if kind in ("step", "decay_step") else (B, H, L, d)
    x["q"] = normal(*shape, scale=d ** -0.5)
    x["k"] = normal(*shape)
    x["v"] = normal(*shape)
    if kind == "backward":
        x["dO"] = normal(*shape, scale=d ** -0.5)
    if kind in ("step", "decay_step") or case["state"]:
        if kind.startswith("decay"):
            x["sk"] = normal(B, H, S, d, scale=0.7, dtype=torch.float32)
            x["sv"] = normal(B, H, S, d, scale=0.7, dtype=torch.float32)
        else:
            for n in ("sk", "sv"):
                x[n] = normal(B, H, 2, M, d, scale=16.0, dtype=torch.float32)
                x[n][:, :, 1, 0].zero_()  # the sine of mode 0
    if kind == "backward" and case["state"]:
        x["gk"] = normal(B, H, 2, M, d, scale=0.05, dtype=torch.float32)
        x["gv"] = normal(B, H, 2, M, d, scale=0.05, dtype=torch.float32)
        x["gk"][:, :, 1, 0].zero_()
        x["gv"][:, :, 1, 0].zero_()
    if case["rows"]:
        x["pos"] = torch.randint(0, 2 * case["t0"] + 1, (B,), generator=g, device=DEV, dtype=torch.int64)
    return x


def prepare(case, seed):
    x = _inputs(case, seed)
    kind, M, S = case["kind"], case["M"], case["S"]
    T = _periods(case)
    st = {"case": case, "x": x, "T": T, "ws": None}
    if not case["keep"]:
        return st
    # The workspace that the program keeps from call to call, sized by the library, and its first call,
    # which leaves the tables there.
    p = bla.make_params(case["B"], case["H"], case["L"], case["d"], M, S, _dtype(case), case["t0"],
                        phase_anchor=case["anchor"])
    size = {"forward": bla.workspace_size, "backward": bla.backward_workspace_size,
            "step": bla.step_workspace_size, "decay_step": bla.step_workspace_size,
            "decay_forward": bla.decay_workspace_size, "layer": bla.layer_workspace_size}[kind]
    st["ws"] = torch.empty(max(size(p), 1), dtype=torch.uint8, device=DEV)
    if kind == "forward":
        bla.forward(x["q"], x["k"], x["v"], T, M, S, t0=case["t0"], state_k=x.get("sk"), state_v=x.get("sv"),
                    workspace=st["ws"], phase_anchor=case["anchor"])
    elif kind == "step":  # one row is enough: the tables do not depend on the batch
        row = [x[n][:1].clone() for n in ("q", "k", "v", "sk", "sv")]
        bla.step(*row[:3], T, M, S, *row[3:], t0=case["t0"], workspace=st["ws"], phase_anchor=case["anchor"])
    return st


def run(state):
    case, x, T, ws = state["case"], state["x"], state["T"], state["ws"]
    kind, M, S, t0, keep = case["kind"], case["M"], case["S"], case["t0"], case["keep"]
    if kind == "forward":
        return bla.forward(x["q"], x["k"], x["v"], T, M, S, t0=t0, state_k=x.get("sk"), state_v=x.get("sv"),
                           workspace=ws, phase_anchor=case["anchor"], reuse_tables=keep)
    if kind == "backward":
        return bla.backward(x["q"], x["k"], x["v"], x["dO"], T, M, S, t0=t0, state_k=x.get("sk"),
                            state_v=x.get("sv"), dstate_k=x.get("gk"), dstate_v=x.get("gv"), workspace=ws)
    if kind == "step":
        o = bla.step(x["q"], x["k"], x["v"], T, M, S, x["sk"], x["sv"], pos=x.get("pos"), t0=t0, workspace=ws,
                     phase_anchor=case["anchor"], reuse_tables=keep)
        return o, x["sk"], x["sv"]
    if kind == "decay_step":
        o = bla.decay_step(x["q"], x["k"], x["v"], T, M, S, x["sk"], x["sv"], pos=x.get("pos"), t0=t0,
                           workspace=ws)
        return o, x["sk"], x["sv"]
    if kind == "decay_forward":
        return bla.decay_forward(x["q"], x["k"], x["v"], T, M, S, t0=t0, slot_k=x.get("sk"), slot_v=x.get("sv"),
                                 workspace=ws)
    return bla.layer_forward(x["x"], x["w_qkv"], x["w_o"], T, case["H"], M, S, t0=t0, workspace=ws)


# ------------------------------------------------------------------------ the same in float64

def _grid(M, S, T, dev):
    """Interpolation weights A, B [S, M] at the slot lags s T / S, and the slots' first positions."""
    m = torch.arange(M, dtype=torch.int64, device=dev)
    s = torch.arange(S, dtype=torch.int64, device=dev)
    c = torch.full((M,), 2.0 / (2 * M - 1), dtype=F64, device=dev)
    c[0] = 1.0 / (2 * M - 1)
    ph = 2 * math.pi * ((s[:, None] * m[None, :]) % S).to(F64) / S
    return c * ph.cos(), c * ph.sin(), torch.round(s.to(F64) * T / S)


def _operator(q, k, v, T, M, S, t0, anchor, zk, zv, block):
    """One head over L tokens in float64: outputs [L, d] and the final states [2, M, d].  Within a block
    that starts from state Z, Z_j = exp(i m w j) (Z + sum_{i <= j} exp(-i m w i) x_i)."""
    L, d = q.shape
    dev = q.device
    A, Bm, first = _grid(M, S, T, dev)
    w = 2 * math.pi / T * torch.arange(M, dtype=F64, device=dev)
    sgn, outs = (-1.0 if anchor else 1.0), []
    for b0 in range(0, L, block):
        n = min(block, L - b0)
        j = torch.arange(1, n + 1, dtype=F64, device=dev)
        co, si = torch.cos(j[:, None] * w), torch.sin(j[:, None] * w)

        def sums(z, x):
            return (z[0] + torch.cumsum(co[:, :, None] * x[:, None, :], 0),
                    z[1] - torch.cumsum(si[:, :, None] * x[:, None, :], 0))

        x = slice(b0, b0 + n)
        kc, ks = sums(zk, k[x])
        vc, vs = sums(zv, v[x])
        a, b = (kc * q[x][:, None, :]).sum(-1), (ks * q[x][:, None, :]).sum(-1)
        if anchor:  # exp(-i m w (p - j)): one phase for the block
            ph = -w * float(t0 + b0 - 1)
            tc, ts = torch.cos(ph)[None, :], torch.sin(ph)[None, :]
        else:
            tc, ts = co, si
        z = (tc * a - ts * b) @ A.T + sgn * ((ts * a + tc * b) @ Bm.T)
        p = (t0 + b0 + torch.arange(n, dtype=F64, device=dev))
        z = (z / math.sqrt(d)).masked_fill(p[:, None] < first[None, :], -math.inf)
        P = torch.softmax(z, -1)
        X, Y = P @ A, sgn * (P @ Bm)
        outs.append(((tc * X + ts * Y)[:, :, None] * vc + (tc * Y - ts * X)[:, :, None] * vs).sum(1))

        def last(c, s):
            return torch.stack([co[-1][:, None] * c[-1] - si[-1][:, None] * s[-1],
                                si[-1][:, None] * c[-1] + co[-1][:, None] * s[-1]])

        zk, zv = last(kc, ks), last(vc, vs)
    return torch.cat(outs), zk, zv


def _heads(case, q, k, v, sk, sv):
    """_operator over every head: outputs [B, H, L, d] and states [B, H, 2, M, d]."""
    B, H, L, d, M, S = (case[x] for x in ("B", "H", "L", "d", "M", "S"))
    block = max(1, (1 << 25) // (M * d))
    o = torch.empty(B, H, L, d, dtype=F64, device=DEV)
    fk = torch.empty(B, H, 2, M, d, dtype=F64, device=DEV)
    fv = torch.empty_like(fk)
    zero = torch.zeros(2, M, d, dtype=F64, device=DEV)
    for b in range(B):
        for h in range(H):
            z = [zero if t is None else t[b, h].to(F64) for t in (sk, sv)]
            o[b, h], fk[b, h], fv[b, h] = _operator(
                q[b, h].to(F64), k[b, h].to(F64), v[b, h].to(F64), _periods(case)[h], M, S, case["t0"],
                case["anchor"], *z, block)
    return o, fk, fv


def _exact_backward(case, x):
    B, H, M, S = (case[n] for n in ("B", "H", "M", "S"))
    shape = (B, H, 2, M, case["d"])
    grads = [torch.empty(x[n].shape, dtype=F64, device=DEV) for n in ("q", "k", "v")]
    grads += [torch.empty(shape, dtype=F64, device=DEV) for _ in range(2)]
    zero = torch.zeros(shape[2:], dtype=F64, device=DEV)
    for b in range(B):
        for h in range(H):
            t = [x[n][b, h].to(F64).requires_grad_() for n in ("q", "k", "v")]
            z = [(x[n][b, h].to(F64) if n in x else zero.clone()).requires_grad_() for n in ("sk", "sv")]
            with torch.enable_grad():
                o, fk, fv = _operator(*t, _periods(case)[h], M, S, case["t0"], False, *z, 1 << 30)
                loss = (o * x["dO"][b, h].to(F64)).sum()
                if "gk" in x:
                    loss = loss + (fk * x["gk"][b, h].to(F64)).sum() + (fv * x["gv"][b, h].to(F64)).sum()
                for out, g in zip(grads, torch.autograd.grad(loss, t + z)):
                    out[b, h] = g
    return tuple(grads)


def _exact_step(case, x):
    """One token per row from the given states, some rows at a time."""
    B, H, d, M, S = (case[n] for n in ("B", "H", "d", "M", "S"))
    pos = x["pos"] if "pos" in x else torch.full((B,), case["t0"], dtype=torch.int64, device=DEV)
    T = torch.tensor(_periods(case), dtype=F64, device=DEV)
    A, Bm, _ = _grid(M, S, 1.0, DEV)
    first = torch.round(torch.arange(S, dtype=F64, device=DEV) * T[:, None] / S)          # [H, S]
    w = 2 * math.pi / T[:, None] * torch.arange(M, dtype=F64, device=DEV)                 # [H, M]
    o = torch.empty(B, H, d, dtype=F64, device=DEV)
    sk, sv = (torch.empty(B, H, 2, M, d, dtype=F64, device=DEV) for _ in range(2))
    for b in range(0, B, 64):
        r = slice(b, min(b + 64, B))
        q, k, v = (x[n][r].to(F64) for n in ("q", "k", "v"))

        def push(z, t):
            z = z.to(F64)
            co, si = torch.cos(w)[..., None], torch.sin(w)[..., None]
            return co * z[:, :, 0] - si * z[:, :, 1] + t[:, :, None], si * z[:, :, 0] + co * z[:, :, 1]

        kc, ks = push(x["sk"][r], k)
        vc, vs = push(x["sv"][r], v)
        a, c = (kc * q[:, :, None]).sum(-1), (ks * q[:, :, None]).sum(-1)
        if case["anchor"]:
            ph = -w * pos[r].to(F64)[:, None, None]
            tc, ts, sgn = torch.cos(ph), torch.sin(ph), -1.0
        else:
            tc, ts, sgn = torch.ones_like(a), torch.zeros_like(a), 1.0
        z = (tc * a - ts * c) @ A.T + sgn * ((ts * a + tc * c) @ Bm.T)
        z = (z / math.sqrt(d)).masked_fill(pos[r].to(F64)[:, None, None] < first, -math.inf)
        P = torch.softmax(z, -1)
        X, Y = P @ A, sgn * (P @ Bm)
        o[r] = ((tc * X + ts * Y)[..., None] * vc + (tc * Y - ts * X)[..., None] * vs).sum(2)
        sk[r, :, 0], sk[r, :, 1], sv[r, :, 0], sv[r, :, 1] = kc, ks, vc, vs
    return o, sk, sv


def _exact_decay(case, x, step):
    """The state-decay form, token by token."""
    B, H, d, M, S = (case[n] for n in ("B", "H", "d", "M", "S"))
    L = 1 if step else case["L"]
    T = torch.tensor(_periods(case), dtype=F64, device=DEV)[:, None]
    tau = torch.arange(S, dtype=F64, device=DEV) * T / S
    first = torch.round(tau)
    pos0 = x["pos"] if "pos" in x else torch.full((B,), case["t0"], dtype=torch.int64, device=DEV)
    q, k, v = (x[n].to(F64).view(B, H, L, d) for n in ("q", "k", "v"))
    K, V = ((x[n].to(F64) if n in x else torch.zeros(B, H, S, d, dtype=F64, device=DEV)) for n in ("sk", "sv"))
    c = torch.full((M,), 2.0 / (2 * M - 1), dtype=F64, device=DEV)
    c[0] = 1.0 / (2 * M - 1)
    m = torch.arange(M, dtype=F64, device=DEV)
    o = torch.empty(B, H, L, d, dtype=F64, device=DEV)
    rows = pos0 if "pos" in x else pos0[:1]  # one gate for the whole batch where it has one position
    for t in range(L):
        p = (rows + t).to(F64)[:, None, None]
        g = (torch.cos(2 * math.pi / T[..., None] * (p - tau)[..., None] * m) * c).sum(-1)
        gs = g[..., None]
        K = torch.lerp(K, k[:, :, t, None], gs)
        V = torch.lerp(V, v[:, :, t, None], gs)
        z = (K * q[:, :, t, None]).sum(-1) / math.sqrt(d)
        P = torch.softmax(z.masked_fill(p < first, -math.inf), -1)
        o[:, :, t] = (P[..., None] * V).sum(2)
    return (o[:, :, 0] if step else o), K, V


@torch.no_grad()
def exact(case, seed):
    x, kind = _inputs(case, seed), case["kind"]
    B, H, L, d, M = (case[n] for n in ("B", "H", "L", "d", "M"))
    if kind == "forward":
        # passes over [L, M, d] float64 sums at some TB/s
        return _heads(case, x["q"], x["k"], x["v"], x.get("sk"), x.get("sv"))
    if kind == "backward":
        return _exact_backward(case, x) if L * M * d <= 1 << 26 else None
    if kind == "step":
        return _exact_step(case, x)
    if kind.startswith("decay"):
        return _exact_decay(case, x, kind == "decay_step")
    qkv = (x["x"].to(F64) @ x["w_qkv"].to(F64)).view(B, L, 3, H, d).permute(2, 0, 3, 1, 4)
    o, fk, fv = _heads(case, *qkv, None, None)
    return o.permute(0, 2, 1, 3).reshape(B, L, H * d) @ x["w_o"].to(F64), fk, fv
