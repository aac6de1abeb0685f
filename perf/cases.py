"""The performance cases of the hybrid-attention layer: what is measured.

A case is one pass through the public entry points of
``paper_2607_24788_amd.glide`` (``state_init``, ``prefill``, ``decode_step``)
at a size of this repository's own workloads, or a drawn one of the same
ranges.  ``exact`` gives the same pass in float64 from the definition of the
layer, in plain torch.

Fields of a case:
  op      "prefill": a prompt into a fresh state (state_init, then prefill);
          "extend": the next tokens of sequences that already hold ``history``
          tokens (chunked serving prefill); "decode": one token per sequence
  calls   "stack": one call over every layer; "layer": one call per layer, as
          a model makes them that interleaves attention with its other blocks
  layers, batch, hq, hkv, d, df, dtype, phi, gated, per_head, chunk: the stack
  w_lo, w_hi   windows, rising geometrically over the layers
  t_lo, t_hi   tokens per sequence: the prompt's or the appended ones
          (prefill, extend), or the context before the step (decode)
  history      tokens held before an "extend"
  scale   standard deviation of q and k ("d": 1/sqrt(d), the repository's
          workloads; "1": unit scale, scores of standard deviation 1)
"""
import math

import torch

from paper_2607_24788_amd import glide

PHI = {"relu": glide.PHI_RELU, "elu1": glide.PHI_ELU1, "softmax": glide.PHI_SOFTMAX}
DTYPE = {"fp32": torch.float32, "bf16": torch.bfloat16}
GATE_LO = -0.4       # log-gates are uniform in [GATE_LO, 0]
FOLD_PERIOD = 8      # decode writes S, z back once per this many steps (W > 0)

BASE = {"op": "prefill", "calls": "stack", "layers": 1, "batch": 1, "hq": 32, "hkv": 8, "d": 128, "df": 128,
        "w_lo": 512, "w_hi": 512, "t_lo": 8192, "t_hi": 8192, "history": 0, "dtype": "bf16", "phi": "relu",
        "gated": False, "per_head": False, "chunk": 0, "scale": "d"}
SMALL = {"hq": 4, "hkv": 4, "d": 64, "df": 64, "w_lo": 64, "w_hi": 64, "dtype": "fp32"}


def _case(name, **kw):
    c = dict(BASE, **kw)
    c["name"] = name
    return c


def listed():
    return [
        # the single fp32 layer, the smallest calls: a prompt of 512 tokens,
        # and a token after it (latency and launches are all there is)
        _case("prefill_fp32_layer", t_lo=512, t_hi=512, **SMALL),
        _case("decode_fp32_layer", op="decode", t_lo=512, t_hi=512, **SMALL),
        # one chat session of an 8B-shaped model, 8K context: the prompt and a
        # decode step over the whole stack (windows rising 16 .. 2048), and
        # the call that its longest-window layer makes inside a model
        _case("prefill_8b_b1_stack", layers=32, w_lo=16, w_hi=2048),
        _case("decode_8b_b1_stack", op="decode", layers=32, w_lo=16, w_hi=2048),
        _case("decode_8b_b1_layer", op="decode", w_lo=2048, w_hi=2048),
        # a serving batch of 32 ragged sequences of 16K .. 32K tokens, windows
        # 64 .. 4096: one decode step in one call, and layer by layer as a
        # model makes it; and the prompts through one long-window layer
        _case("decode_8b_b32_stack", op="decode", layers=32, batch=32, w_lo=64, w_hi=4096, t_lo=16384, t_hi=32768),
        _case("decode_8b_b32_layers", op="decode", calls="layer", layers=32, batch=32, w_lo=64, w_hi=4096,
              t_lo=16384, t_hi=32768),
        _case("prefill_8b_b32_w4096", batch=32, w_lo=4096, w_hi=4096, t_lo=16384, t_hi=32768),
        # long prompts through one layer at the window of most layers, scores
        # of unit deviation; and through a layer that is fully linear
        _case("prefill_8b_4x32k_w512", batch=4, t_lo=32768, t_hi=32768, scale="1"),
        _case("prefill_8b_4x32k_linear", batch=4, w_lo=0, w_hi=0, t_lo=32768, t_hi=32768),
        # chunked serving: odd numbers of new tokens onto 16K of history, with
        # the softmax feature map (the paper's default kernel)
        _case("extend_8b_b8_w1000", op="extend", batch=8, w_lo=1000, w_hi=1000, t_lo=301, t_hi=2047, history=16001,
              phi="softmax"),
        # a 70B-shaped layer (8 query heads per KV head), gated state, an odd
        # long window, 8 sequences
        _case("decode_70b_b8_gated", op="decode", batch=8, hq=64, w_lo=8191, w_hi=8191, t_lo=32768, t_hi=65536,
              gated=True, scale="1"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A single-layer call of the same ranges (odd sizes among them)."""
    c = dict(BASE)
    c["op"] = rng.choice(["prefill", "extend", "decode", "decode"])
    c["hq"], c["hkv"], c["d"], c["df"] = rng.choice(
        [(32, 8, 128, 128), (32, 8, 128, 128), (64, 8, 128, 128), (32, 8, 128, 64), (8, 8, 128, 128), (4, 4, 64, 64),
         (8, 2, 64, 64)])
    c["batch"] = _log_int(rng, 1, 32)
    c["w_lo"] = c["w_hi"] = 0 if rng.random() < 0.1 else _log_int(rng, 16, 8192)
    c["phi"] = rng.choice(["relu", "relu", "elu1", "softmax"])
    c["gated"] = rng.random() < 0.15
    c["per_head"] = rng.random() < 0.15
    c["scale"] = rng.choice(["d", "1"])
    if rng.random() < 0.2:
        c["dtype"] = "fp32"
    if c["op"] == "decode":
        c["t_hi"] = _log_int(rng, 512, 32768)
    elif c["op"] == "extend":
        c["history"] = _log_int(rng, 64, 16384)
        c["t_hi"] = _log_int(rng, 33, 4096)
        c["chunk"] = rng.choice([0, 0, 32, 128])
    else:
        c["t_hi"] = _log_int(rng, 512, 32768)
        c["chunk"] = rng.choice([0, 0, 0, 32, 128, 256])
    # at most 128K tokens in all, 16K of them in fp32
    most = max(33, (16384 if c["dtype"] == "fp32" else 131072) // c["batch"])
    c["t_hi"] = min(c["t_hi"], most)
    c["history"] = min(c["history"], most)
    c["t_lo"] = max(1, int(c["t_hi"] * rng.choice([0.5, 0.8, 1.0])))
    return c


# ---------------------------------------------------------------------------
# sizes

def _windows(c):
    L, lo, hi = c["layers"], c["w_lo"], c["w_hi"]
    return [int(round(lo * (hi / lo) ** (l / (L - 1)))) if L > 1 else hi for l in range(L)]


def _lens(c):
    """Tokens per sequence, spread evenly over [t_lo, t_hi] in a fixed mixed order."""
    B, lo, hi = c["batch"], c["t_lo"], c["t_hi"]
    if B == 1:
        return [hi]
    step = next(s for s in (5, 7, 3, 11, 13) if math.gcd(s, B) == 1)
    return [lo + round((hi - lo) * ((b * step) % B) / (B - 1)) for b in range(B)]


def _glide(c):
    return glide.Glide(c["layers"], c["batch"], c["hq"], c["hkv"], c["d"], c["df"], _windows(c),
                       dtype=DTYPE[c["dtype"]], phi=PHI[c["phi"]], gated=c["gated"], per_head_phi=c["per_head"])


def work(case):
    c = case
    e = 2 if c["dtype"] == "bf16" else 4
    d, Df, Hq, Hkv, B = c["d"], c["df"], c["hq"], c["hkv"], c["batch"]
    state = Hkv * (Df * d + Df) * 4
    bytes_, flops = 0.0, 0.0
    for W in _windows(c):
        bytes_ += d * Df * e * (Hkv if c["per_head"] else 1)
        for n in _lens(c):
            if c["op"] == "decode":
                w = min(W, n)
                # window K/V, the new token in and into the ring, q in, O out,
                # the state read, and written once per fold period
                bytes_ += (2 * w + 4) * Hkv * d * e + 2 * Hq * d * e
                bytes_ += state * (1 + (1 / FOLD_PERIOD if W > 0 else 1))
                flops += 4 * Hq * d * w + 4 * Hq * d * Df + 2 * Hkv * d * Df
            else:
                p0 = c["history"]
                keys = sum_min(p0, n, W)
                bytes_ += (2 * n + 2 * min(W, p0)) * Hkv * d * e + 2 * n * Hq * d * e
                bytes_ += 2 * min(W, n) * Hkv * d * e + 2 * state
                # phi of q and k, the band's two products, state update and read-out
                flops += 2 * ((Hq + Hkv) * n * d * Df + 2 * Hq * d * keys + Hkv * n * Df * d + Hq * n * Df * d)
    return {"bytes": bytes_, "flops": flops}


def sum_min(p0, n, W):
    """sum over positions t in [p0, p0 + n) of min(t + 1, W)."""
    a = max(0, min(n, W - p0))       # positions whose window is not full yet
    return a * p0 + a * (a + 1) // 2 + (n - a) * W


# ---------------------------------------------------------------------------
# inputs

def _inputs(c, seed):
    """Every tensor of the case, from its seed: phi weights, the history's
    k, v and log-gates (one layer's, shared by every layer of the stack), the
    new tokens' q, k, v and log-gates per layer."""
    g = torch.Generator(device="cuda")
    g.manual_seed(1000003 * int(seed) + 17)
    dt, L, d, Df = DTYPE[c["dtype"]], c["layers"], c["d"], c["df"]
    s = d ** -0.5

    def normal(shape, scale):
        x = torch.empty(shape, dtype=dt, device="cuda")
        flat, step = x.view(-1), 1 << 28
        for i in range(0, flat.numel(), step):
            n = min(step, flat.numel() - i)
            flat[i:i + n] = torch.randn(n, generator=g, device="cuda").mul_(scale)
        return x

    def gates(shape):
        return torch.rand(shape, generator=g, device="cuda") * GATE_LO if c["gated"] else None

    qk = 1.0 if c["scale"] == "1" else s
    lens = _lens(c)
    hist = {"decode": lens, "extend": [c["history"]] * c["batch"], "prefill": [0] * c["batch"]}[c["op"]]
    new = [1] * c["batch"] if c["op"] == "decode" else lens
    T, H = sum(new), sum(hist)
    x = {"hist": hist, "new": new}
    x["wf"] = normal((L, c["hkv"], d, Df) if c["per_head"] else (L, d, Df), s)
    x["q"] = normal((L, T, c["hq"], d), qk)
    x["k"] = normal((L, T, c["hkv"], d), qk)
    x["v"] = normal((L, T, c["hkv"], d), s)
    x["gate"] = gates((L, T, c["hkv"]))
    x["hk"] = normal((H, c["hkv"], d), qk)
    x["hv"] = normal((H, c["hkv"], d), s)
    x["hgate"] = gates((H, c["hkv"]))
    return x


def _cu(lens):
    cu = [0]
    for n in lens:
        cu.append(cu[-1] + n)
    return cu


class State:
    pass


def prepare(case, seed):
    c = case
    x = _inputs(c, seed)
    st = State()
    st.op, st.by_layer, st.layers = c["op"], c["calls"] == "layer", c["layers"]
    st.g = g = _glide(c)
    st.state = g.new_state()
    g.state_init(st.state)
    st.ws = g.new_workspace(sum(x["new"]) if c["op"] != "decode" else 0)
    st.wf, st.q, st.k, st.v, st.gate = x["wf"], x["q"], x["k"], x["v"], x["gate"]
    st.out = torch.empty_like(st.q)
    st.cu, st.chunk = _cu(x["new"]), c["chunk"]
    if sum(x["hist"]):  # the tokens the sequences hold already
        T = sum(x["hist"])
        ws = g.new_workspace(T)
        q = torch.zeros((T, c["hq"], c["d"]), dtype=st.q.dtype, device="cuda")
        out = torch.empty_like(q)
        for l in range(c["layers"]):
            g.prefill(st.state, st.wf[l], q, x["hk"], x["hv"], _cu(x["hist"]), out, ws, layer0=l, n_layers=1,
                      log_gates=x["hgate"])
    # the state beside the outputs: S and z of every layer, then the K and V
    # rings (of the 31 longest windows in a deeper stack: at most 64 tensors)
    es = st.q.element_size()
    st.views = []
    for l in range(c["layers"]):
        lay = g.layout(l)
        st.views.append(st.state[lay.s_offset:lay.z_offset + c["batch"] * c["hkv"] * c["df"] * 4].view(torch.float32))
    for l in range(max(0, c["layers"] - 31), c["layers"]):
        lay = g.layout(l)
        if lay.ring_slots:
            n = c["batch"] * c["hkv"] * lay.ring_slots * c["d"] * es
            st.views.append(st.state[lay.kring_offset:lay.vring_offset + n].view(st.q.dtype))
    return st


def run(state):
    st = state
    if st.op == "decode":
        if st.by_layer:
            for l in range(st.layers):
                st.g.decode_step(st.state, st.wf[l], st.q[l], st.k[l], st.v[l], st.out[l], st.ws, layer0=l, n_layers=1,
                                 log_gates=None if st.gate is None else st.gate[l])
        else:
            st.g.decode_step(st.state, st.wf, st.q, st.k, st.v, st.out, st.ws, log_gates=st.gate)
    else:
        if st.op == "prefill":
            st.g.state_init(st.state)
        st.g.prefill(st.state, st.wf, st.q, st.k, st.v, st.cu, st.out, st.ws, chunk=st.chunk, log_gates=st.gate)
    return [st.out] + st.views


def tolerance(case):
    """Relative 2-norm.  bf16: four times the path's own distance from
    ``exact`` (0.0015 .. 0.0023 over the cases and drawn ones; rounding of the
    weights and of the output).  fp32: scores of unit deviation reach 30 in
    the exponent, where one rounding is 1e-6 of the weight (2e-7 seen at the
    workloads' scale)."""
    return {"rel": 8e-3} if case["dtype"] == "bf16" else {"rel": 5e-6}


# ---------------------------------------------------------------------------
# the layer in float64

def _phi(c, x, wf):
    y = x @ wf
    if c["phi"] == "relu":
        return y.clamp_min(0)
    if c["phi"] == "elu1":
        return torch.where(y > 0, y + 1, y.clamp_max(0).exp())
    return torch.softmax(y, -1)


def _sequence(c, W, wf, q, k, v, gate, p0):
    """One sequence: outputs [Hq][n][d] of the last n = q.shape[1] tokens, and
    S, z after them.  q [Hq][n][d]; k, v [Hkv][p][d]; gate [Hkv][p] or None;
    wf [Hkv or 1][d][Df]; all float64."""
    Hkv, p, d = k.shape
    G, n = q.shape[0] // Hkv, q.shape[1]
    tau = d ** -0.5
    fk = _phi(c, k, wf)
    fq = _phi(c, q.view(Hkv, G * n, d), wf).view(Hkv, G, n, -1)
    q = q.view(Hkv, G, n, d)
    cum = torch.cumsum(gate, 1) if gate is not None else None
    out = torch.empty((Hkv, G, n, d), dtype=torch.float64, device=k.device)
    C = 512
    S = torch.zeros((Hkv, fk.shape[-1], d), dtype=torch.float64, device=k.device)
    z = torch.zeros((Hkv, fk.shape[-1]), dtype=torch.float64, device=k.device)
    done, ref = 0, None  # S, z: tokens [0, done), decayed to position ref

    def fold(end, at):
        nonlocal S, z, done, ref
        at = max(at, 0)
        if cum is not None and ref is not None:
            f = (cum[:, at] - cum[:, ref]).exp()
            S, z = S * f[:, None, None], z * f[:, None]
        if end > done:
            w = fk[:, done:end]
            if cum is not None:
                w = w * (cum[:, at, None] - cum[:, done:end]).exp()[:, :, None]
            S = S + w.transpose(1, 2).contiguous() @ v[:, done:end]
            z = z + w.sum(1)
            done = end
        ref = at

    for i0 in range(0, n, C):
        i1 = min(n, i0 + C)
        t0, t1 = p0 + i0, p0 + i1
        t = torch.arange(t0, t1, device=k.device)
        # the state before the block's first linear-set change, decayed to t0
        fold(max(0, t0 - W), t0)
        fqb = fq[:, :, i0:i1].reshape(Hkv, G * (i1 - i0), -1)
        if cum is not None:
            fac = (cum[:, t0:t1] - cum[:, t0:t0 + 1]).exp()[:, None, :, None]
            fac = fac.expand(Hkv, G, i1 - i0, 1).reshape(Hkv, -1, 1)
        else:
            fac = 1.0
        num, den = (fqb @ S) * fac, (fqb @ z[:, :, None]) * fac
        j0, j1 = max(0, t0 - W), max(0, t1 - W)  # tokens that join within the block
        if j1 > j0:
            j = torch.arange(j0, j1, device=k.device)
            a = fqb @ fk[:, j0:j1].transpose(1, 2).contiguous()
            a = a.view(Hkv, G, i1 - i0, j1 - j0) * (j[None, :] <= t[:, None] - W)
            if cum is not None:
                a = a * (cum[:, t0:t1, None] - cum[:, None, j0:j1]).clamp_max(0).exp()[:, None]
            a = a.view(Hkv, -1, j1 - j0)
            num, den = num + a @ v[:, j0:j1], den + a.sum(-1, keepdim=True)
        if W > 0:
            b0 = max(0, t0 - W + 1)
            j = torch.arange(b0, t1, device=k.device)
            s = (q[:, :, i0:i1].reshape(Hkv, -1, d) @ k[:, b0:t1].transpose(1, 2).contiguous()) * tau
            s = s.view(Hkv, G, i1 - i0, t1 - b0)
            s = s.masked_fill(~((j[None, :] <= t[:, None]) & (j[None, :] > t[:, None] - W)), -math.inf)
            m = s.amax(-1, keepdim=True)
            e = (s - m).exp_().view(Hkv, -1, t1 - b0)
            f = (-m).exp().view(Hkv, -1, 1)
            num, den = e @ v[:, b0:t1] + num * f, e.sum(-1, keepdim=True) + den * f
        out[:, :, i0:i1] = torch.where(den > 0, num / den, 0.0).view(Hkv, G, i1 - i0, d)
    fold(max(0, p - W), p - 1)
    return out.view(Hkv * G, n, d), S, z


def _ring_raw(x, R, d, values):
    """[..][R][d] by slot -> the ring's storage order (include/glide.h)."""
    s, col = torch.arange(R, device=x.device)[:, None], torch.arange(d, device=x.device)[None, :]
    o = s % 32
    if values:
        at = ((col // 16 * 4 + o // 8) * 16 + col % 16) * 8 + o % 8
    else:
        at = ((((o // 4) % 2 * (d // 32) + col // 32) * 4 + (col // 8) % 4) * 16 + 4 * (o // 8) + o % 4) * 8 + col % 8
    at = (s // 32) * 32 * d + at
    y = torch.empty_like(x).view(*x.shape[:-2], R * d)
    y[..., at.reshape(-1)] = x.reshape(*x.shape[:-2], R * d)
    return y


def _ring(c, W, xs, p0, p, values):
    """Ring contents after a prefill to p0 tokens and then on to p: each call
    leaves its last W tokens in their slots.  xs [Hkv][p][d]."""
    R = (W + 8 + 31) // 32 * 32
    r = torch.zeros((xs.shape[0], R, c["d"]), dtype=torch.float64, device=xs.device)
    for lo, hi in ((0, p0), (p0, p)):
        j = torch.arange(max(lo, hi - W), hi, device=xs.device)
        r[:, j % R] = xs[:, j]
    return _ring_raw(r, R, c["d"], values)


def exact(case, seed):
    c = case
    if work(c)["flops"] > 8e13:
        return None  # minutes in float64
    x = _inputs(c, seed)
    cu, hcu = _cu(x["new"]), _cu(x["hist"])
    f64 = lambda y: y.double().transpose(0, 1).contiguous()  # [tokens][heads][..] -> [heads][tokens][..]  # noqa: E731
    out = torch.empty(x["q"].shape, dtype=torch.float64, device="cuda")
    states, rings = [], []
    for l, W in enumerate(_windows(c)):
        wf = x["wf"][l].double().view(-1, c["d"], c["df"]).expand(c["hkv"], c["d"], c["df"]).contiguous()
        S, z, kr, vr = [], [], [], []
        for b in range(c["batch"]):
            h, i = slice(hcu[b], hcu[b + 1]), slice(cu[b], cu[b + 1])
            k = f64(torch.cat([x["hk"][h], x["k"][l, i]]))
            v = f64(torch.cat([x["hv"][h], x["v"][l, i]]))
            gate = None
            if c["gated"]:
                gate = torch.cat([x["hgate"][h], x["gate"][l, i]]).double().t().contiguous()
            o, s_, z_ = _sequence(c, W, wf, f64(x["q"][l, i]), k, v, gate, x["hist"][b])
            out[l, i] = o.transpose(0, 1)
            S.append(s_)
            z.append(z_)
            if W:
                p0, p = x["hist"][b], x["hist"][b] + x["new"][b]
                kr.append(_ring(c, W, k, p0, p, False))
                vr.append(_ring(c, W, v, p0, p, True))
        # after a decode step S, z leave out the tokens still pending, up to
        # FOLD_PERIOD of them by a schedule of the library's own
        states.append(torch.cat([torch.stack(S).view(-1), torch.stack(z).view(-1)]) if c["op"] != "decode" else None)
        if W and l >= c["layers"] - 31:
            rings.append(torch.cat([torch.stack(kr).view(-1), torch.stack(vr).view(-1)]))
    return [out] + states + rings
