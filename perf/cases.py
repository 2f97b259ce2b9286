"""Workloads that the speed of this framework is judged by: the calls its users make, at the sizes they make them.

``listed()`` names the standing cases, ``draw(rng)`` makes further ones of the same ranges, ``prepare`` / ``run`` set a
case up and make one pass through the public entry points, ``exact`` gives the outputs in 64-bit torch, ``work`` the
bytes and operations a pass cannot do without and ``tolerance`` how far two correct implementations may differ.
"""
import math

import torch

import paper_2503_05447_amd as lsm

NONE, HEAD, SCALAR, VECTOR = lsm.DECAY_NONE, lsm.DECAY_HEAD, lsm.DECAY_SCALAR, lsm.DECAY_VECTOR
DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}


def _case(name, op, **kw):
    """op: "step", "delta_step" (one decoded token), "fwd" (prefill), "train" (forward + backward), "delta_train".
    kind: decay kind; law: distribution of the log-decay; tokens_first: [B,T,H,d] order; lengths: comma-separated
    sequence lengths of a packed batch ("" = B sequences of T tokens); init: the sequence starts from a state."""
    c = dict(name=name, op=op, B=1, H=16, T=1, d_k=128, d_v=128, dtype="bf16", kind=SCALAR, law="default",
             tokens_first=False, lengths="", init=False, gated=False)
    c.update(kw)
    return c


def listed():
    return [
        # A chat-sized decode batch of a Mamba2-style layer (16 heads of 128): one token for each of 4 sequences.
        # Latency of a single launch.
        _case("decode_scalar_b4", "step", B=4),
        # A serving batch decoding with a Gated DeltaNet layer: 128 sequences, the whole state read and written.
        _case("decode_gated_delta_b128", "delta_step", B=128, gated=True),
        # Basic linear attention in fp32 on a short text, forward only: the numerics-check call (configuration 1).
        _case("bla_f32_short", "fwd", B=1, H=2, T=256, d_k=64, d_v=64, dtype="f32", kind=NONE),
        # Serving prefill: unequal prompts packed on one token axis, in the order a fused QKV projection leaves them.
        _case("prefill_packed", "fwd", T=9373, tokens_first=True, lengths="1,37,64,511,900,1283,2481,4096"),
        # Prefill of one prompt by a model with 64-wide heads.
        _case("prefill_heads64", "fwd", H=32, T=1777, d_k=64, d_v=64, tokens_first=True),
        # Training steps of a layer (forward keeps its states for the backward call): configurations 2, 3, 4 and 5.
        _case("train_head_t2048", "train", B=8, T=2048, kind=HEAD),
        _case("train_scalar_t8192", "train", B=4, T=8192),
        _case("train_vector_t4096", "train", B=4, T=4096, d_v=256, kind=VECTOR),
        # A long-document shard: the state comes in from the shard before and its gradient goes back there.
        _case("train_long_carried", "train", H=32, T=65536, law="strong", init=True),
        # Training step of a DeltaNet layer.
        _case("train_delta_t2048", "delta_train", B=16, T=2048),
        # Training in fp32 (the reference precision for debugging a run), a length that is no multiple of a chunk.
        _case("train_f32_t2047", "train", B=4, T=2047, dtype="f32"),
        # Training step of a gated-linear-attention layer in its usual head shape: keys of 64, values of 128.
        _case("train_gla_heads64", "train", B=4, H=8, T=2048, d_k=64, d_v=128, kind=VECTOR),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the ranges the listed ones stand for: every entry point, decay kind, element type and head shape."""
    op = rng.choice(["step", "delta_step", "fwd", "fwd", "train", "train", "train", "delta_train"])
    if op in ("step", "delta_step"):
        dims = (128, 128) if rng.random() < 0.5 else (rng.choice([64, 128, 256]), rng.choice([64, 128, 256]))
        H = rng.choice([4, 8, 16, 32])
        B = _log_int(rng, 4, max(5, min(256, (1 << 26) // (H * dims[0] * dims[1]))))
        gated = rng.random() < 0.5
        return _case("", op, B=B, H=H, d_k=dims[0], d_v=dims[1], dtype=rng.choice(["bf16", "bf16", "f32"]),
                     kind=(SCALAR if gated else NONE) if op == "delta_step" else rng.choice([NONE, HEAD, SCALAR, VECTOR]),
                     gated=gated)
    tokens_first = rng.random() < 0.5
    H = rng.choice([2, 4, 8, 16, 32])
    if op == "delta_train":
        T = _log_int(rng, 100, 16384)
        B = _log_int(rng, 1, max(1, min(32, (1 << 19) // (H * T))))
        gated = rng.random() < 0.5
        return _case("", op, B=B, H=H, T=T, gated=gated, kind=SCALAR if gated else NONE, tokens_first=tokens_first,
                     init=rng.random() < 0.3)
    kind = rng.choice([NONE, HEAD, SCALAR, SCALAR, VECTOR])
    # half of the draws are bf16 with 128-wide keys, the shape of the model series; the others spread over the rest
    if rng.random() < 0.5:
        dtype, d_k, d_v, most = "bf16", 128, rng.choice([128, 128, 256]), 1 << 19
    else:
        dtype, d_k, d_v, most = rng.choice(["bf16", "f32"]), rng.choice([64, 64, 128]), rng.choice([64, 128]), 1 << 16
    T = _log_int(rng, 64, 16384)
    lengths = ""
    B = _log_int(rng, 1, max(1, min(32, most // (H * T))))
    if T * H > most:
        T = most // H
    if op == "fwd" and T >= 256 and rng.random() < 0.5:
        B, n = 1, rng.randint(2, 12)
        cuts = sorted(rng.sample(range(1, T), n - 1))
        lengths = ",".join(str(b - a) for a, b in zip([0] + cuts, cuts + [T]))
    return _case("", op, B=B, H=H, T=T, d_k=d_k, d_v=d_v, dtype=dtype, kind=kind, tokens_first=tokens_first,
                 lengths=lengths, init=rng.random() < 0.3)


# ---- inputs ------------------------------------------------------------------------------------------------------

def _inputs(case, seed):
    """q, k, v, d_o, decays, strengths and edge states from the seed alone, with the values the layers see: q and k of
    length about 1 (exactly 1 for the delta rule's keys), data-dependent log-decays, write strengths in (0, 1)."""
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev).manual_seed(seed)
    B, H, T, dk, dv = (case[n] for n in ("B", "H", "T", "d_k", "d_v"))
    delta = case["op"].startswith("delta")
    step = case["op"] in ("step", "delta_step")
    lead = (B, H) if step else ((B, T, H) if case["tokens_first"] else (B, H, T))
    dt = DTYPES[case["dtype"]]

    def normal(*shape):
        return torch.randn(shape, generator=gen, device=dev)
    x = {"q": (normal(*lead, dk) / dk ** 0.5).to(dt)}
    k = normal(*lead, dk)
    x["k"] = (torch.nn.functional.normalize(k, dim=-1) if delta else k / dk ** 0.5).to(dt)
    del k
    x["v"] = (normal(*lead, dv) / (1 if delta else dk ** 0.5)).to(dt)
    x["d_o"] = normal(*lead, dv).to(dt) if case["op"].endswith("train") else None
    shift = 4.0 if case["law"] == "strong" else 3.0
    g = None
    if case["kind"] == HEAD:
        g = -torch.exp2(-(5.0 + 8.0 * torch.arange(H, device=dev) / H))
    elif case["kind"] == SCALAR:
        g = -torch.nn.functional.softplus(normal(*lead) + shift)
    elif case["kind"] == VECTOR:
        g = torch.nn.functional.logsigmoid(normal(*lead, dk)) / 16
    x["g"] = g
    x["b"] = torch.sigmoid(normal(*lead)) if delta else None
    x["beta"] = x["b"].clone() if delta and not case["gated"] else None
    n_seq = len(_lengths(case)) or B
    x["state"] = normal(n_seq, H, dk, dv) * 0.1 if step or case["init"] else None
    x["d_final"] = normal(n_seq, H, dk, dv) * 0.1 if case["init"] and case["op"].endswith("train") else None
    return x


def _lengths(case):
    return [int(n) for n in case["lengths"].split(",")] if case["lengths"] else []


def prepare(case, seed):
    s = _inputs(case, seed)
    s["case"] = case
    layout = lsm.LAYOUT_BTHD if case["tokens_first"] else lsm.LAYOUT_BHTD
    s["layout"] = layout
    s["cu"] = None
    if case["lengths"]:
        cu = [0]
        for n in _lengths(case):
            cu.append(cu[-1] + n)
        s["cu"] = torch.tensor(cu, dtype=torch.int32, device="cuda")
    # training programs keep one workspace that the forward call's states travel through to the backward call
    if case["op"] == "train":
        s["ws"] = lsm.lsm_chunk_workspace(s["q"], s["k"], s["v"], s["g"], case["kind"], layout=layout)
    elif case["op"] == "delta_train":
        s["ws"] = lsm.lsm_delta_workspace(s["q"], s["k"], s["v"], s["g"], layout=layout)
    return s


def run(s):
    case, kind, layout = s["case"], s["case"]["kind"], s["layout"]
    q, k, v, g = s["q"], s["k"], s["v"], s["g"]
    if case["op"] == "step":
        o = lsm.lsm_step(q, k, v, g, kind, s["state"])
        return {"o": o, "state": s["state"]}
    if case["op"] == "delta_step":
        o = lsm.lsm_delta_step(q, k, v, s["state"], g, s["beta"], s["b"])
        return {"o": o, "state": s["state"]}
    if case["op"] == "fwd":
        o, final = lsm.lsm_chunk_fwd(q, k, v, g, kind, init_state=s["state"], layout=layout, cu_seqlens=s["cu"])
        return {"o": o, "final_state": final}
    if case["op"] == "train":
        o, final = lsm.lsm_chunk_fwd(q, k, v, g, kind, init_state=s["state"], workspace=s["ws"], layout=layout,
                                     save_states=True)
        r = lsm.lsm_chunk_bwd(q, k, v, g, kind, s["d_o"], init_state=s["state"], d_final_state=s["d_final"],
                              workspace=s["ws"], layout=layout, states_saved=True)
    else:
        o, final = lsm.lsm_delta_fwd(q, k, v, g, s["beta"], s["b"], init_state=s["state"], workspace=s["ws"],
                                     layout=layout, save_states=True)
        r = lsm.lsm_delta_bwd(q, k, v, s["d_o"], g, s["beta"], s["b"], init_state=s["state"],
                              d_final_state=s["d_final"], workspace=s["ws"], layout=layout, states_saved=True)
    r = {n: t for n, t in r.items() if t is not None}
    return dict(r, o=o, final_state=final)


# ---- what a pass cannot do without ----------------------------------------------------------------------------------

def work(case):
    """Inputs read once and outputs written once; multiply-adds of the token recurrence (a state update and a read-out
    per token, their four adjoint products in the backward, one more product each for the delta rule's erase term)."""
    B, H, T, dk, dv = (case[n] for n in ("B", "H", "T", "d_k", "d_v"))
    e = 2 if case["dtype"] == "bf16" else 4
    heads, delta, train = B * H, case["op"].startswith("delta"), case["op"].endswith("train")
    if case["op"] in ("step", "delta_step"):
        T = 1
    tok = heads * T
    per_token = {NONE: 0, HEAD: 0, SCALAR: 1, VECTOR: dk}[case["kind"]]
    if delta:
        per_token += 1 if case["gated"] else 2
    states = (len(_lengths(case)) or B) * H * dk * dv * 4
    byt = tok * ((2 * dk + 2 * dv) * e + 4 * per_token)                          # q, k, v, decays -> o
    if case["op"] in ("step", "delta_step"):
        byt += 2 * states
    else:
        byt += states * (2 if case["init"] else 1)
    flops = tok * 2 * dk * dv * (3 if delta else 2)
    if train:
        byt += tok * ((4 * dk + 3 * dv) * e + 8 * per_token) + states * (3 if case["init"] else 1)
        flops += tok * 2 * dk * dv * (6 if delta else 4)
    return {"bytes": int(byt), "flops": int(flops)}


def tolerance(case):
    """About four times the largest distance to ``exact`` seen on the listed cases and a few dozen drawn ones.

    bf16 outputs carry their own rounding (2-norm 1.7e-3; 2.3e-3 for dk, dv under a weak decay, where a per-chunk
    state gradient is held in bf16; single elements up to 2e-2 of the result's root mean square there).  fp32: the
    decay gradient, a sum of terms that cancel, is the furthest off (2-norm 4.1e-6, elements 2.3e-5); a decode step
    is one short sum (2e-7, 2e-6)."""
    step = case["op"] in ("step", "delta_step")
    if case["dtype"] == "f32":
        return {"rel": 1e-6, "max": 1e-5} if step else {"rel": 1.6e-5, "max": 1e-4}
    return {"rel": 7e-3, "max": 1.6e-2} if step else {"rel": 9e-3, "max": 8e-2}


# ---- the same results in 64 bits ------------------------------------------------------------------------------------

CHUNK = 64   # the factored decays exp(b), exp(-b) of a block stay far inside the range of 64-bit floats


def _blocks(x, n):
    """[R,T,d] -> [R,n,CHUNK,d], zero-padded."""
    R, T, d = x.shape
    return torch.nn.functional.pad(x, (0, 0, 0, n * CHUNK - T)).reshape(R, n, CHUNK, d)


def _recurrence(q, k, v, g, m0, beta=None, b=None):
    """o, final state of M_t = a_t (I - beta_t k^T k) M_{t-1} + b_t k^T v, o = q M, for R sequences [R,T,d] in blocks."""
    R, T, dk = q.shape
    dv = v.shape[-1]
    n = -(-T // CHUNK)
    delta = b is not None
    q, k, v = _blocks(q, n), _blocks(k, n), _blocks(v, n)
    g = torch.zeros(R, T, 1, dtype=q.dtype, device=q.device) if g is None else g
    cum = _blocks(g, n).cumsum(2)
    last = cum[:, :, -1:]
    qe, ke, kd = q * cum.exp(), k * (-cum).exp(), k * (last - cum).exp()
    keep = last.exp().transpose(2, 3)                                             # [R,n,dk or 1,1]
    A = torch.tril(qe @ ke.transpose(2, 3))
    if delta:
        b = _blocks(b, n)
        be = torch.ones_like(b) if beta is None else _blocks(beta, n)
        L = torch.tril(be * ((k * cum.exp()) @ ke.transpose(2, 3)), -1)
        eye = torch.eye(CHUNK, dtype=q.dtype, device=q.device)
        inv, power = eye - L, L @ L                                               # (I + L)^-1, L nilpotent
        for _ in range(int(math.log2(CHUNK)) - 1):
            inv, power = inv @ (eye + power), power @ power
        uhat, what = inv @ (b * v), inv @ (be * k * cum.exp())
        kdt, S, us, states = kd.transpose(2, 3), m0, [], []
        for c in range(n):
            u = uhat[:, c] - what[:, c] @ S
            states.append(S)
            us.append(u)
            S = keep[:, c] * S + kdt[:, c] @ u
        v = torch.stack(us, 1)
    else:
        U = kd.transpose(2, 3) @ v
        S, states = m0, []
        for c in range(n):
            states.append(S)
            S = keep[:, c] * S + U[:, c]
    o = A @ v + qe @ torch.stack(states, 1)
    return o.reshape(R, n * CHUNK, dv)[:, :T], S


def _rows(x, tokens_first):
    """[B,H,T,...] or [B,T,H,...] -> [B*H,T,d] in 64 bits."""
    x = x.double()
    if tokens_first:
        x = x.transpose(1, 2)
    x = x.reshape(x.shape[0] * x.shape[1], x.shape[2], -1)
    return x


def exact(case, seed):
    x = _inputs(case, seed)
    B, H, T, dk, dv = (case[n] for n in ("B", "H", "T", "d_k", "d_v"))
    dev = x["q"].device
    if case["op"] in ("step", "delta_step"):
        q, k, v, M = (x[n].double() for n in ("q", "k", "v", "state"))
        a = torch.ones((), dtype=torch.float64, device=dev) if x["g"] is None else x["g"].double().exp()
        a = {NONE: a, HEAD: a.reshape(-1)[:, None, None], SCALAR: a[..., None, None] if a.dim() else a,
             VECTOR: a[..., None]}[case["kind"]]
        if case["op"] == "delta_step":
            be = 1.0 if x["beta"] is None else x["beta"].double()[..., None, None]
            kM = (k[..., None] * M).sum(-2, keepdim=True)
            M = a * (M - be * k[..., None] * kM) + x["b"].double()[..., None, None] * k[..., None] * v[..., None, :]
        else:
            M = a * M + k[..., None] * v[..., None, :]
        return {"o": (q[..., None] * M).sum(-2), "state": M}
    tf, train = case["tokens_first"], case["op"].endswith("train")
    g = x["g"]
    if case["kind"] == HEAD:   # one value per head, its gradient summed over batch and tokens
        g = g.reshape(1, 1, H).expand(B, T, H) if tf else g.reshape(1, H, 1).expand(B, H, T)
    names = [n for n, t in (("q", x["q"]), ("k", x["k"]), ("v", x["v"]), ("g", g), ("beta", x["beta"]), ("b", x["b"]))
             if t is not None]
    full = {n: _rows(t, tf) for n, t in dict(x, g=g).items() if n in names}
    bounds = [(0, T)]
    if case["lengths"]:
        cu = [0]
        for n in _lengths(case):
            cu.append(cu[-1] + n)
        bounds = list(zip(cu, cu[1:]))
    n_seq = len(bounds) if case["lengths"] else B
    m0 = (torch.zeros(n_seq, H, dk, dv, device=dev) if x["state"] is None else x["state"]).double().reshape(-1, dk, dv)
    out = {"o": torch.empty(B * H, T, dv, dtype=torch.float64, device=dev), "final_state": torch.empty_like(m0)}
    if train:
        d_o = _rows(x["d_o"], tf)
        d_fin = torch.zeros_like(m0) if x["d_final"] is None else x["d_final"].double().reshape(-1, dk, dv)
        for n in names:
            out["d_" + n] = torch.empty_like(full[n])
        out["d_init_state"] = torch.empty_like(m0)
    step = max(1, (1 << 20) // T)   # recurrences at a time: bounds the states that are held
    for s, (lo, hi) in enumerate(bounds):
        for r0 in range(0, B * H, step):
            r1 = min(B * H, r0 + step)
            e = slice(s * H + r0, s * H + r1) if case["lengths"] else slice(r0, r1)
            leaf = {n: t[r0:r1, lo:hi].detach().requires_grad_(train) for n, t in full.items()}
            start = m0[e].detach().requires_grad_(train)
            o, fin = _recurrence(leaf["q"], leaf["k"], leaf["v"], leaf.get("g"), start, leaf.get("beta"), leaf.get("b"))
            if train:
                grads = torch.autograd.grad((o * d_o[r0:r1, lo:hi]).sum() + (fin * d_fin[e]).sum(),
                                            [leaf[n] for n in names] + [start])
                for n, t in zip(names, grads):
                    out["d_" + n][r0:r1, lo:hi] = t
                out["d_init_state"][e] = grads[-1]
            out["o"][r0:r1, lo:hi], out["final_state"][e] = o.detach(), fin.detach()

    def back(t, like):
        t = t.reshape(B, H, T, -1)
        t = t.transpose(1, 2) if tf else t
        return t.reshape(like).contiguous()
    res = {"o": back(out["o"], x["v"].shape), "final_state": out["final_state"].reshape(n_seq, H, dk, dv)}
    if train:
        for n in ("q", "k", "v"):
            res["d" + n] = back(out["d_" + n], x[n].shape)
        res["d_init_state"] = out["d_init_state"].reshape(n_seq, H, dk, dv)
        if g is not None:
            dg = out["d_g"].reshape(B, H, T).sum((0, 2)) if case["kind"] == HEAD else back(out["d_g"], x["g"].shape)
            res["d_log_alpha" if case["op"] == "delta_train" else "dg"] = dg
        for n in ("beta", "b"):
            if n in names:
                res["d_" + n] = back(out["d_" + n], x[n].shape)
    return res
