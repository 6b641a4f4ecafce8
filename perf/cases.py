"""Performance cases of the W4A8 layers, called as a serving program calls them.

Every case goes through the functions of paper_2608_12932_amd on tensors that
are already on the GPU, with a workspace that the program keeps; outputs are
allocated by the calls.  The sizes are those of the decoder layer that the
package's inputs describe (hidden 4096, 32 query heads on 8 kv heads of 128,
MLP width 12288), of the streaming window (views x frames x tokens) and of the
action head (6 trajectories of 128 values).

Kinds of cases:
  linear     one projection: bf16 x (quantized inside the call) or int8 codes
  swiglu     the fused gate+up projection with its gated activation
  norm       RMSNorm + int8 quantize of the tokens in front of a projection
  attention  streaming prefill attention of the newest frame over the window
  flow       one action solve: Euler steps with the cached velocity
  layers     consecutive decoder layers: norm, qkv, o, norm, gate+up, down
"""
import math

import torch

import paper_2608_12932_amd as w

HIDDEN, MLP, HEAD_DIM = 4096, 12288, 128
QKV = 6144
GROUP = 128
# name -> (K, N) of the layer's projections
MATS = {"qkv": (HIDDEN, QKV), "o": (HIDDEN, HIDDEN), "gate_up": (HIDDEN, 2 * MLP), "down": (MLP, HIDDEN)}
EPS = 1e-6
LARGEST_OPS = 2 * 2048 * 24576 * 4096


def listed():
    return [
        # one token of plain decoding, the smallest projection of the layer
        dict(name="decode_o_m1", kind="linear", M=1, K=4096, N=4096, group=True, i8=False, f32=False),
        # verification of a 16-token draft block: the widest projection
        dict(name="verify_gate_up_m16", kind="linear", M=16, K=4096, N=24576, group=False, i8=False, f32=False),
        # verification of a short draft: the longest reduction
        dict(name="verify_down_m4", kind="linear", M=4, K=12288, N=4096, group=False, i8=False, f32=False),
        # several draft blocks at once, codes already made by the norm prologue
        dict(name="verify_qkv_m48", kind="linear", M=48, K=4096, N=6144, group=True, i8=True, f32=False),
        # streaming prefill of the new frame's tokens
        dict(name="prefill_qkv_m1024", kind="linear", M=1024, K=4096, N=6144, group=False, i8=False, f32=False),
        # a short prefill chunk through the longest reduction
        dict(name="prefill_down_m256", kind="linear", M=256, K=12288, N=4096, group=True, i8=False, f32=False),
        # a whole window's prefill through the widest projection: the largest call
        dict(name="prefill_gate_up_m2048", kind="linear", M=2048, K=4096, N=24576, group=True, i8=False, f32=False),
        # the gated MLP projection on a ragged number of new-frame tokens
        dict(name="prefill_swiglu_m777", kind="swiglu", M=777, K=4096, N=24576, group=False, i8=False, f32=False),
        # the norm in front of a projection during prefill
        dict(name="norm_m1024", kind="norm", M=1024, K=4096),
        # streaming attention of one layer: 4 views x 4 frames x 192 tokens
        dict(name="attention_4x4x192", kind="attention", V=4, F=4, T=192, shift=1, H=32, Hkv=8),
        # one action solve: 8 steps, 4 of them reusing the cached velocity
        dict(name="flow_6x128", kind="flow", B=6, n=128, steps=8, reuse=4),
        # draft verification through the projections of two whole layers
        dict(name="layers_m16", kind="layers", M=16, L=2, group=True),
    ]


def draw(rng):
    def log_int(lo, hi):
        return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))

    kind = rng.choices(["linear", "swiglu", "norm", "attention", "flow", "layers"], [7, 2, 1, 2, 1, 1])[0]
    if kind in ("linear", "swiglu"):
        if kind == "swiglu":
            K, N = HIDDEN, 32 * log_int(64, 768)
        elif rng.random() < 0.5:
            K, N = MATS[rng.choice(sorted(MATS))]
        else:  # other widths and shards of the same projections
            K, N = 128 * log_int(8, 96), 16 * log_int(64, 1536)
        M = log_int(1, 2048)
        while 2 * M * N * K > LARGEST_OPS:
            M //= 2
        return dict(kind=kind, M=M, K=K, N=N, group=rng.random() < 0.5, i8=rng.random() < 0.3, f32=rng.random() < 0.15)
    if kind == "norm":
        return dict(kind="norm", M=log_int(1, 4096), K=128 * log_int(8, 96))
    if kind == "attention":
        H, Hkv = rng.choice([(8, 2), (16, 4), (32, 8), (16, 16), (28, 4)])
        F = rng.randint(2, 6)
        return dict(kind="attention", V=rng.randint(1, 6), F=F, T=rng.randint(16, 256), shift=rng.randrange(F), H=H, Hkv=Hkv)
    if kind == "flow":
        steps = rng.randint(4, 16)
        return dict(kind="flow", B=log_int(1, 4096), n=log_int(32, 2048), steps=steps, reuse=rng.randrange(steps))
    return dict(kind="layers", M=log_int(1, 512), L=1, group=rng.random() < 0.5)


# ---------------------------------------------------------------- inputs


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _tokens(g, M, K):
    """Activations: N(0, 1) with 1 % of the channels 20 times larger, in bf16."""
    x = torch.randn(M, K, generator=g, device="cuda")
    x[:, torch.randperm(K, generator=g, device="cuda")[: round(0.01 * K)]] *= 20.0
    return x.to(torch.bfloat16)


def _weight(g, N, K, group):
    W = torch.randint(-8, 8, (N, K), generator=g, device="cuda", dtype=torch.int8)
    if group:
        s = (torch.rand(K // GROUP, N, generator=g, device="cuda") * 0.015 + 0.005).to(torch.float16)
    else:
        s = torch.rand(N, generator=g, device="cuda") * 0.015 + 0.005
    return W, s


def _gamma(g, K):
    return (1.0 + 0.1 * torch.randn(K, generator=g, device="cuda")).to(torch.bfloat16)


def _linear_inputs(c, seed):
    g = _gen(seed)
    x = _tokens(g, c["M"], c["K"])
    W, s = _weight(g, c["N"], c["K"], c["group"])
    return x, W, s


def _norm_inputs(c, seed):
    g = _gen(seed)
    return _tokens(g, c["M"], c["K"]), _gamma(g, c["K"])


def _attention_inputs(c, seed):
    """Queries: the newest frame of every view; cache: each view's frames in a
    ring, slot (f + shift) % F holding frame f."""
    g = _gen(seed)
    V, F, T = c["V"], c["F"], c["T"]
    Nq, Nk = V * T, V * F * T
    t = torch.arange(T, device="cuda", dtype=torch.int32)
    pos_k = torch.empty(V, F, T, device="cuda", dtype=torch.int32)
    for v in range(V):
        for f in range(F):
            pos_k[v, (f + c["shift"]) % F] = (v * F + f) * T + t
    pos_q = torch.cat([(v * F + F - 1) * T + t for v in range(V)])
    q = torch.randn(c["H"], Nq, HEAD_DIM, generator=g, device="cuda").to(torch.bfloat16)
    k = torch.randn(c["Hkv"], Nk, HEAD_DIM, generator=g, device="cuda").to(torch.bfloat16)
    v = torch.randn(c["Hkv"], Nk, HEAD_DIM, generator=g, device="cuda").to(torch.bfloat16)
    inv = 1e6 ** (-torch.arange(HEAD_DIM // 2, device="cuda", dtype=torch.float64) * 2 / HEAD_DIM)
    ang = torch.arange(Nk, device="cuda", dtype=torch.float64)[:, None] * inv
    return q, k, v, pos_q, pos_k.reshape(-1), ang.cos().float(), ang.sin().float()


def _flow_inputs(c, seed):
    """The noise start and one velocity per evaluated step."""
    g = _gen(seed)
    x0 = torch.randn(c["B"], c["n"], generator=g, device="cuda")
    n_eval = c["steps"] - c["reuse"]
    base = torch.randn(c["B"], c["n"], generator=g, device="cuda") * 2
    vs = [(base + 0.3 * torch.randn(c["B"], c["n"], generator=g, device="cuda")).to(torch.bfloat16) for _ in range(n_eval)]
    return x0, vs


def _flow_repeats(c):
    """Steps per evaluated velocity: an evaluation and the reused steps after it."""
    head = (c["steps"] - c["reuse"] + 1) // 2
    rep = [1] * (c["steps"] - c["reuse"])
    rep[head - 1] += c["reuse"]
    return rep


def _layers_inputs(c, seed):
    g = _gen(seed)
    x = _tokens(g, c["M"], HIDDEN)
    layers = []
    for _ in range(c["L"]):
        layers.append(dict(attn=_tokens(g, c["M"], HIDDEN), g1=_gamma(g, HIDDEN), g2=_gamma(g, HIDDEN),
                           **{m: _weight(g, MATS[m][1], MATS[m][0], c["group"]) for m in sorted(MATS)}))
    return x, layers


# ---------------------------------------------------------------- the calls


def _mode(group):
    return w.SCALE_GROUP_F16 if group else w.SCALE_CHANNEL_F32


def prepare(case, seed):
    c = case
    st = dict(c=c, ws=w.Workspace())
    if c["kind"] in ("linear", "swiglu"):
        x, W, s = _linear_inputs(c, seed)
        st.update(x=x, sx=None, wp=w.w4a8_pack_weights(W), s=s, mode=_mode(c["group"]),
                  out=w.OUT_F32 if c["f32"] else w.OUT_BF16)
        if c["i8"]:
            st["x"], st["sx"] = w.w4a8_quantize_act(x)
    elif c["kind"] == "norm":
        st["x"], st["gamma"] = _norm_inputs(c, seed)
    elif c["kind"] == "attention":
        st["args"] = _attention_inputs(c, seed)
    elif c["kind"] == "flow":
        st["x0"], st["vs"] = _flow_inputs(c, seed)
        st["cache"] = torch.zeros_like(st["vs"][0])
        st["fresh"] = w.w4a8_flow_schedule(c["steps"], c["reuse"])
    else:
        st["x"], layers = _layers_inputs(c, seed)
        st["mode"] = _mode(c["group"])
        st["layers"] = [{k: (w.w4a8_pack_weights(v[0]), v[1]) if k in MATS else v for k, v in d.items()} for d in layers]
    return st


def _run_flow(st):
    c = st["c"]
    x, cache = st["x0"].clone(), st["cache"]
    dt, stats, i, e = 1.0 / c["steps"], [], 0, 0
    fresh = st["fresh"]
    while i < c["steps"]:
        n = 1
        while i + n < c["steps"] and not fresh[i + n]:
            n += 1
        s = w.w4a8_flow_step(x, st["vs"][e], cache, dt, stats=e > 0, repeat=n)
        if s is not None:
            stats.append(s)
        i, e = i + n, e + 1
    return x, cache, stats


def _run_layers(st):
    mode, ws, h, outs = st["mode"], st["ws"], st["x"], []
    for d in st["layers"]:
        q, sx = w.w4a8_rmsnorm_quantize_act(h, d["g1"], EPS)
        qkv = w.w4a8_linear(q, *d["qkv"], QKV, x_scale=sx, scale_mode=mode, workspace=ws)
        o = w.w4a8_linear(d["attn"], *d["o"], HIDDEN, scale_mode=mode, workspace=ws)
        q, sx = w.w4a8_rmsnorm_quantize_act(o, d["g2"], EPS)
        m = w.w4a8_linear_swiglu(q, *d["gate_up"], 2 * MLP, x_scale=sx, scale_mode=mode, workspace=ws)
        h = w.w4a8_linear(m, *d["down"], HIDDEN, scale_mode=mode, workspace=ws)
        outs += [qkv, o, h]
    return outs


def run(state):
    st, kind = state, state["c"]["kind"]
    if kind == "linear":
        return w.w4a8_linear(st["x"], st["wp"], st["s"], st["c"]["N"], x_scale=st["sx"], scale_mode=st["mode"],
                             out_kind=st["out"], workspace=st["ws"])
    if kind == "swiglu":
        return w.w4a8_linear_swiglu(st["x"], st["wp"], st["s"], st["c"]["N"], x_scale=st["sx"], scale_mode=st["mode"],
                                    out_kind=st["out"], workspace=st["ws"])
    if kind == "norm":
        return w.w4a8_rmsnorm_quantize_act(st["x"], st["gamma"], EPS)
    if kind == "attention":
        return w.w4a8_stream_attention(*st["args"], HEAD_DIM ** -0.5, workspace=st["ws"])
    if kind == "flow":
        return _run_flow(st)
    return _run_layers(st)


# ---------------------------------------------------------------- work, tolerance


def _linear_work(M, K, N, group, i8, out_bytes, out_cols=None):
    cols = N if out_cols is None else out_cols
    scales = N * K // GROUP * 2 if group else N * 4
    x = M * K + 4 * M if i8 else 2 * M * K
    return N * K // 2 + scales + x + M * cols * out_bytes, 2 * M * N * K


def work(case):
    c = case
    if c["kind"] in ("linear", "swiglu"):
        cols = c["N"] // 2 if c["kind"] == "swiglu" else c["N"]
        b, f = _linear_work(c["M"], c["K"], c["N"], c["group"], c["i8"], 4 if c["f32"] else 2, cols)
    elif c["kind"] == "norm":
        b, f = c["M"] * c["K"] * 3 + 4 * c["M"] + 2 * c["K"], 6 * c["M"] * c["K"]
    elif c["kind"] == "attention":
        V, F, T, H, Hkv = c["V"], c["F"], c["T"], c["H"], c["Hkv"]
        # query t of view v sees all keys at positions up to its own
        pairs = sum((v * F + F - 1) * T * T + T * (T + 1) // 2 for v in range(V))
        Nq, Nk = V * T, V * F * T
        b = 2 * H * Nq * HEAD_DIM * 2 + 2 * Hkv * Nk * HEAD_DIM * 2 + 4 * (Nq + Nk) + 2 * Nk * HEAD_DIM // 2 * 4
        f = 4 * HEAD_DIM * pairs * H
    elif c["kind"] == "flow":
        n_eval, elems = c["steps"] - c["reuse"], c["B"] * c["n"]
        # the start, one state pass and one velocity per evaluation
        b, f = elems * (8 + n_eval * (8 + 4)), elems * (2 * c["steps"] + 8 * n_eval)
    else:
        b = f = 0
        for m, i8, ob, cols in (("qkv", True, 2, None), ("o", False, 2, None), ("gate_up", True, 2, MLP), ("down", False, 2, None)):
            lb, lf = _linear_work(c["M"], *MATS[m], c["group"], i8, ob, cols)
            b, f = b + lb, f + lf
        b, f = c["L"] * (b + 2 * (3 * c["M"] * HIDDEN)), c["L"] * f
    return {"bytes": b, "flops": f}


def tolerance(case):
    k = case["kind"]
    if k in ("linear", "swiglu"):
        # integer sums are exact and the scaling is fp32; the output's type rounds
        return {"rel": 1e-6} if case["f32"] else {"rel": 7e-3}
    if k == "norm":  # fp32 scales; a code moves by one where a value sits on a tie
        return {"rel": 1e-6, "differ": 1e-4}
    if k == "attention":  # bf16 weights of the value sum and a bf16 output
        return {"rel": 9e-3}
    if k == "flow":  # two fp32 roundings a step; the sums are fp64
        return {"rel": 1e-6}
    # bf16 between the projections: a moved rounding moves codes of the next
    return {"rel": 2e-2}


# ---------------------------------------------------------------- 64-bit reference


def _codes(x):
    """Per-token codes as the format defines them: fp32 scale absmax / 127,
    round half to even of the fp32 quotient."""
    x = x.float()
    a = x.abs().amax(1, keepdim=True)
    s = a / torch.full_like(a, 127.0)  # a tensor divides; a Python number would multiply by its reciprocal
    q = torch.where(s > 0, torch.round(x / torch.where(s > 0, s, torch.ones_like(s))), torch.zeros_like(x))
    return q.double(), s.double()


def _exact_linear(x, W, s, group):
    q, sx = _codes(x)
    Wd = W.double()
    if group:
        Wd *= s.double().t().repeat_interleave(GROUP, 1)
        return (q @ Wd.t()) * sx
    return (q @ Wd.t()) * sx * s.double()


def _silu_mul(y):
    F = y.shape[1] // 2
    return torch.nn.functional.silu(y[:, :F]) * y[:, F:]


def _norm64(x, gamma):
    x = x.double()
    return x * torch.rsqrt(x.square().mean(1, keepdim=True) + EPS) * gamma.double()


def _exact_attention(args):
    q, k, v, pos_q, pos_k, cos, sin = args
    half = HEAD_DIM // 2

    def rotate(x, pos):  # rotate-half in fp32, held in bf16 as the model holds it
        a, b = x[..., :half].float(), x[..., half:].float()
        c, s = cos[pos.long()], sin[pos.long()]
        return torch.cat([a * c - b * s, b * c + a * s], -1).to(torch.bfloat16).double()

    qr, kr, v = rotate(q, pos_q), rotate(k, pos_k), v.double()
    seen = pos_k[None, :] <= pos_q[:, None]
    out = []
    for h in range(q.shape[0]):
        hk = h // (q.shape[0] // k.shape[0])
        s = (qr[h] @ kr[hk].t()) * HEAD_DIM ** -0.5
        out.append(torch.softmax(s.masked_fill(~seen, -math.inf), 1) @ v[hk])
    return torch.stack(out)


def exact(case, seed):
    c = case
    if c["kind"] in ("linear", "swiglu"):
        y = _exact_linear(*_linear_inputs(c, seed), c["group"])
        return y if c["kind"] == "linear" else _silu_mul(y)
    if c["kind"] == "norm":
        h = _norm64(*_norm_inputs(c, seed))
        return None, h.abs().amax(1) / 127.0
    if c["kind"] == "attention":
        return _exact_attention(_attention_inputs(c, seed))
    if c["kind"] == "flow":
        x, vs = _flow_inputs(c, seed)
        x, stats, prev = x.double(), [], None
        for v, n in zip((v.double() for v in vs), _flow_repeats(c)):
            if prev is not None:
                stats.append(torch.stack([(v * prev).sum(1), (v * v).sum(1), (prev * prev).sum(1), (v - prev).square().sum(1)], 1))
            x, prev = x + n * v / c["steps"], v
        return x, prev, stats
    x, layers = _layers_inputs(c, seed)
    h, outs = x, []
    for d in layers:
        qkv = _exact_linear(_norm64(h, d["g1"]), *d["qkv"], c["group"])
        o = _exact_linear(d["attn"], *d["o"], c["group"])
        m = _silu_mul(_exact_linear(_norm64(o, d["g2"]), *d["gate_up"], c["group"]))
        h = _exact_linear(m, *d["down"], c["group"])
        outs += [qkv, o, h]
    return outs
