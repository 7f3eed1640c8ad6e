"""Performance cases of the framework: what a user has it do, timed one pass at a time.

``listed()`` names the fixed cases, ``draw(rng)`` gives another one of the same
ranges, ``prepare`` makes a case's inputs on the GPU, ``run`` takes them once
through the public entry points, and ``exact`` gives the same outputs in 64-bit
torch arithmetic that shares no code with the library.

Kinds of pass:

* ``scan``  - ``bdlru_scan_forward`` then ``bdlru_scan_backward``: the gated scan
  from given pre-activations, one training pass (the benchmark's headline).
* ``layer`` - ``bdlru_forward`` then ``bdlru_backward``: the same with the gate
  projections, one training pass of the BD-LRU layer.
* ``gated`` - ``gated_forward`` then ``gated_backward``: the gated recurrent
  layer core (causal conv, BD-LRU, output gate), one training pass.
* ``prefill`` - ``gated_forward`` alone, h not kept: reading a user's history in
  before serving.
* ``step``  - ``bdlru_step``: one recurrent decode step over a batch of users.
* ``model`` - ``ModelStep.train_step``: loss and gradients of the whole model.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2406_12580_amd import recblr as rb

TAPS = 4  # conv taps of the gated layer
DROPOUT = 0.2  # the rate of the model's benchmark


def listed():
    return [
        # A handful of short histories in fp32: the smallest training call, all latency.
        {"name": "scan_train_small", "kind": "scan", "io": "f32", "B": 4, "L": 50, "D": 64},
        # The paper's training batch: 2048 histories of 200 items, embedding width 64.
        {"name": "scan_train_batch", "kind": "scan", "io": "f32", "B": 2048, "L": 200, "D": 64},
        # Long histories, the benchmark's default workload.
        {"name": "scan_train_long", "kind": "scan", "io": "f32", "B": 256, "L": 2048, "D": 128},
        # Very long histories of few users in bf16: few channels, much sequence.
        {"name": "scan_train_verylong_bf16", "kind": "scan", "io": "bf16", "B": 16, "L": 16384,
         "D": 256},
        # The BD-LRU layer at the long-history shape, weights and all, in fp32.
        {"name": "layer_train_long", "kind": "layer", "io": "f32", "B": 256, "L": 2048, "D": 128},
        # The layer at the very long shape in bf16, the widest weights that are common.
        {"name": "layer_train_verylong_bf16", "kind": "layer", "io": "bf16", "B": 16, "L": 16384,
         "D": 256},
        # Odd batch and length, a width that is no power of two, an initial state.
        {"name": "layer_train_ragged_bf16", "kind": "layer", "io": "bf16", "B": 37, "L": 777,
         "D": 192, "h0": True},
        # The gated layer as the model trains it: batch 2048, length 200, width 2 * 64.
        {"name": "gated_train_batch", "kind": "gated", "io": "f32", "B": 2048, "L": 200, "D": 128},
        # Serving: the histories of 32 users read in, bf16, no backward to follow.
        {"name": "gated_prefill_bf16", "kind": "prefill", "io": "bf16", "B": 32, "L": 1000,
         "D": 256},
        # Decode for a few users at once: one launch's latency.
        {"name": "step_few_bf16", "kind": "step", "io": "bf16", "B": 8, "D": 256},
        # Decode for 65,536 users at once.
        {"name": "step_many_bf16", "kind": "step", "io": "bf16", "B": 65536, "D": 256},
        # One training step of the whole model, MovieLens-1M sizes, dropout and left padding.
        {"name": "model_train_ml1m", "kind": "model", "io": "f32", "B": 2048, "T": 200, "D": 64,
         "V": 3416, "layers": 2},
    ]


# Elements B * L * D of a drawn case, smallest and largest, by kind.
RANGES = {"scan": (4e3, 6.7e7), "layer": (6e4, 6.7e7), "gated": (6e4, 5.2e7),
          "prefill": (3e4, 1.6e7), "step": (5e2, 1.6e7)}


def _spread(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    kind = rng.choice(["scan", "layer", "layer", "gated", "gated", "prefill", "step", "model"])
    if kind == "model":
        D = rng.choice([64, 64, 128])
        rows = _spread(rng, 2000, 2.0e5 if D == 64 else 1.0e5)
        T = int(round(_spread(rng, 20, 200)))
        return {"kind": kind, "io": "f32", "B": max(8, int(rows / T)), "T": T, "D": D,
                "V": int(_spread(rng, 500, 12000)), "layers": rng.choice([1, 2])}
    io = rng.choice(["f32", "bf16"])
    # Widths: the powers of two and multiples of 64 of the configurations, and odd ones.
    D = rng.choice([64, 64, 128, 128, 128, 256, 256, 192, 72, 100])
    lo, hi = RANGES[kind]
    n = _spread(rng, lo, hi)
    if kind == "step":
        return {"kind": kind, "io": io, "B": max(1, int(n / D)), "D": D}
    rows = max(1.0, n / D)
    L = int(_spread(rng, min(20, rows), min(16384, rows)))
    B = max(1, int(rows / L))
    return {"kind": kind, "io": io, "B": B, "L": max(1, L), "D": D,
            "h0": bool(rng.random() < 0.3)}


# ------------------------------------------------------------------ inputs

def _dtype(case):
    return torch.float32 if case["io"] == "f32" else torch.bfloat16


def _normal(g, shape, dtype=torch.float32, scale=1.0):
    return (torch.randn(shape, generator=g, device="cuda") * scale).to(dtype)


def _uniform(g, shape, lo, hi, dtype=torch.float32):
    return (torch.rand(shape, generator=g, device="cuda") * (hi - lo) + lo).to(dtype)


def _lambda(g, D, lo, hi):
    """Lambda from decay bases a ~ U[lo, hi] as the paper initialises it: ln(1 / a - 1)."""
    a = torch.rand(D, generator=g, device="cuda", dtype=torch.float64) * (hi - lo) + lo
    return torch.log(1.0 / a - 1.0).float()


def _model_layout(case):
    """[(name, shape, offset)] of the flat parameters (each tensor at a multiple of 64 floats)."""
    D, E, V = case["D"], 2, case["V"]
    ED = E * D
    one = [("Wx", (ED, D)), ("bx", (ED,)), ("Wz", (ED, D)), ("bz", (ED,)), ("conv_w", (ED, TAPS)),
           ("conv_b", (ED,)), ("Wr", (ED, ED)), ("br", (ED,)), ("Wi", (ED, ED)), ("bi", (ED,)),
           ("lambda", (ED,)), ("Wo", (D, ED)), ("bo", (D,)), ("ln1_g", (D,)), ("ln1_b", (D,)),
           ("W1", (4 * D, D)), ("b1", (4 * D,)), ("W2", (D, 4 * D)), ("b2", (D,)),
           ("ln2_g", (D,)), ("ln2_b", (D,))]
    items = [("emb", (V, D)), ("emb_ln_g", (D,)), ("emb_ln_b", (D,))]
    for l in range(case["layers"]):
        items += [("l%d.%s" % (l, n), s) for n, s in one]
    out, off = [], 0
    for name, shape in items:
        out.append((name, shape, off))
        off += -(-math.prod(shape) // 64) * 64
    return out, off


def _model_inputs(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    layout, total = _model_layout(case)
    flat = torch.zeros(total, device="cuda")
    for name, shape, off in layout:
        n = name.split(".")[-1]
        if n == "lambda":
            v = _lambda(g, shape[0], 0.9, 0.999)
        elif n in ("emb_ln_g", "ln1_g", "ln2_g"):
            v = 1.0 + _uniform(g, shape, -0.1, 0.1)
        elif n == "emb":
            v = _normal(g, shape)
        elif len(shape) == 2:
            v = _normal(g, shape, scale=shape[1] ** -0.5)
        else:
            v = _uniform(g, shape, -0.1, 0.1)
        flat[off:off + math.prod(shape)] = v.reshape(-1)
    B, T, V = case["B"], case["T"], case["V"]
    # Zipf-popular items; rows of 0.655 T to T items, left-padded with id 0.
    pr = 1.0 / torch.arange(1, V, device="cuda", dtype=torch.float64)
    cdf = torch.cumsum(pr / pr.sum(), 0).float()

    def items(shape):
        u = torch.rand(shape, generator=g, device="cuda")
        return (1 + torch.searchsorted(cdf, u).clamp_(max=V - 2)).int()

    ids, targets = items((B, T)), items((B,))
    least = max(1, int(round(0.655 * T)))
    lengths = torch.randint(least, T + 1, (B, 1), generator=g, device="cuda")
    ids[torch.arange(T, device="cuda")[None, :] < T - lengths] = 0
    return flat, ids.contiguous(), targets


def _inputs(case, seed):
    """Named inputs of every kind but the model."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    B, L, D, kind, dt = case["B"], case.get("L", 1), case["D"], case["kind"], _dtype(case)
    # Decay bases: the paper's initialisation, closer to 1 for long histories.
    lo, hi = (0.99, 0.9999) if L > 512 or kind == "step" else (0.9, 0.999)
    s = {"lam": _lambda(g, D, lo, hi), "h0": None}
    if case.get("h0"):
        s["h0"] = _normal(g, (B, D))
    if kind == "scan":
        for n in ("x", "zr", "zi", "dh"):
            s[n] = _normal(g, (B, L, D), dt)
        return s
    for n in ("Wr", "Wi"):
        s[n] = _normal(g, (D, D), dt, D ** -0.5)
    for n in ("br", "bi"):
        s[n] = _uniform(g, (D,), -1.0, 1.0, dt)
    if kind == "step":
        s["x"], s["h_prev"] = _normal(g, (B, D), dt), _normal(g, (B, D))
    elif kind == "layer":
        s["x"], s["dh"] = _normal(g, (B, L, D), dt), _normal(g, (B, L, D), dt)
    else:
        s["hx"], s["hz"] = _normal(g, (B, L, D), dt), _normal(g, (B, L, D), dt)
        s["conv_w"], s["conv_b"] = _normal(g, (D, TAPS), scale=0.5), _normal(g, (D,), scale=0.1)
        if kind == "gated":
            s["dy"] = _normal(g, (B, L, D), dt)
    return s


def prepare(case, seed):
    if case["kind"] != "model":
        return {"case": case, **_inputs(case, seed)}
    flat, ids, targets = _model_inputs(case, seed)
    step = rb.ModelStep(rb.model_dims(case["B"], case["T"], case["D"], V=case["V"],
                                      layers=case["layers"], K=TAPS))
    return {"case": case, "step": step, "params": flat, "ids": ids, "targets": targets,
            "seed": seed}


def run(state):
    s, kind = state, state["case"]["kind"]
    if kind == "scan":
        h, hT = rb.bdlru_scan_forward(s["x"], s["zr"], s["zi"], s["lam"], s["h0"])
        g = rb.bdlru_scan_backward(s["x"], s["zr"], s["zi"], s["lam"], h, s["dh"], s["h0"])
        return {"h": h, "hT": hT, **g}
    if kind == "layer":
        w = (s["Wr"], s["br"], s["Wi"], s["bi"], s["lam"])
        h, hT = rb.bdlru_forward(s["x"], *w, s["h0"])
        g = rb.bdlru_backward(s["x"], *w, h, s["dh"], s["h0"])
        return {"h": h, "hT": hT, **g}
    if kind in ("gated", "prefill"):
        w = (s["conv_w"], s["conv_b"], s["Wr"], s["br"], s["Wi"], s["bi"], s["lam"])
        if kind == "prefill":
            y, _, hT = rb.gated_forward(s["hx"], s["hz"], *w, s["h0"], keep_h=False)
            return {"y": y, "hT": hT}
        y, h, hT = rb.gated_forward(s["hx"], s["hz"], *w, s["h0"])
        g = rb.gated_backward(s["hx"], s["hz"], *w, h, s["dy"], s["h0"])
        return {"y": y, "h": h, "hT": hT, **{k: v for k, v in g.items() if v is not None}}
    if kind == "step":
        return {"h": rb.bdlru_step(s["x"], s["Wr"], s["br"], s["Wi"], s["bi"], s["lam"],
                                   s["h_prev"])}
    loss, grads = s["step"].train_step(s["params"], s["ids"], s["targets"], dropout=DROPOUT,
                                       seed=s["seed"], offset=1, pad_id=0)
    return {"loss": loss, "grads": grads}


# ------------------------------------------------------------------ work and tolerance

def work(case):
    """Each tensor that a call reads or writes, once; the projections' products (the
    backward forms z again, since it isn't handed over) and the gate arithmetic."""
    B, L, D, kind = case["B"], case.get("L", 1), case["D"], case["kind"]
    e = 4 if case["io"] == "f32" else 2
    if kind == "model":
        n, ED, layers = B * case["T"], 2 * D, case["layers"]
        _, total = _model_layout(case)
        # Products per position and layer: input projections, gates, output projection, PFFN;
        # forward, and two products each backward (the gates' z once more).
        mm = 2 * ED * D + 2 * ED * ED + ED * D + 8 * D * D
        flops = 2.0 * n * layers * (3 * mm + 2 * ED * ED) + 6.0 * B * case["V"] * D
        # What a training step keeps of each layer, written once and read once: the layer's
        # input, Hx, Hz, the BD-LRU output, both residual sums, the PFFN pre-activation.
        kept = n * layers * 4.0 * (D + 3 * ED + 2 * D + 4 * D)
        return {"bytes": 2 * kept + 4.0 * n + 8.0 * total, "flops": flops}
    n, w = B * L * D, 2 * D * (D + 1) * e
    if kind == "scan":
        return {"bytes": 12.0 * n * e, "flops": 75.0 * n}
    if kind == "layer":
        return {"bytes": 6.0 * n * e + 2 * w + 8.0 * D * D, "flops": (16.0 * D + 75) * n}
    if kind == "gated":
        return {"bytes": 10.0 * n * e + 2 * w + 8.0 * D * D, "flops": (16.0 * D + 120) * n}
    if kind == "prefill":
        return {"bytes": 3.0 * n * e + w, "flops": (4.0 * D + 40) * n}
    return {"bytes": n * (e + 8.0) + w, "flops": (4.0 * D + 25) * n}


def tolerance(case):
    """About four times the largest error against 64 bits that any output showed: 1.6e-5 in
    fp32 (an initial state's gradient over a long history; 6e-6 otherwise), 2.4e-3 in bf16
    (the rounding of the stored outputs), 2e-7 for one step, 5e-6 over the model's gradients."""
    if case["kind"] == "model":
        return {"rel": 2e-5}
    if case["kind"] == "step":
        return {"rel": 1e-6}
    return {"rel": 6e-5} if case["io"] == "f32" else {"rel": 1e-2}


# ------------------------------------------------------------------ 64-bit reference

def _recur(a, u, h0):
    """h_t = a_t h_{t-1} + u_t over the leading axis."""
    h = torch.empty_like(u)
    prev = torch.zeros_like(u[0]) if h0 is None else h0
    for t in range(u.shape[0]):
        torch.addcmul(u[t], a[t], prev, out=h[t])
        prev = h[t]
    return h


class _Recurrence(torch.autograd.Function):
    """The recurrence with its adjoint delta_t = g_t + a_{t+1} delta_{t+1}."""

    @staticmethod
    def forward(ctx, a, u):
        h = _recur(a, u, None)
        ctx.save_for_backward(a, h)
        return h

    @staticmethod
    def backward(ctx, g):
        a, h = ctx.saved_tensors
        d = _adjoint(a, g)
        da = torch.zeros_like(d)
        da[1:] = d[1:] * h[:-1]
        return da, d


def _adjoint(a, g):
    d = torch.empty_like(g)
    d[-1] = g[-1]
    for t in range(g.shape[0] - 2, -1, -1):
        torch.addcmul(g[t], a[t + 1], d[t + 1], out=d[t])
    return d


def _gates(zr, zi, lam):
    r, i = torch.sigmoid(zr), torch.sigmoid(zi)
    q = torch.nn.functional.softplus(lam) * r
    return r, i, torch.exp(-q), torch.sqrt(-torch.expm1(-2.0 * q))


def _scan64(x, zr, zi, lam, h0, dh=None):
    """h and, given dh, the gradients dx (through beta x), dzr, dzi, dlambda, dh0.
    Sequence tensors are [L][B][D]."""
    r, i, a, s = _gates(zr, zi, lam)
    h = _recur(a, s * i * x, h0)
    if dh is None:
        return h, None
    d = _adjoint(a, dh)
    hp = torch.empty_like(h)
    hp[0] = 0.0 if h0 is None else h0
    hp[1:] = h[:-1]
    dq = -a * (d * hp) + d * x * i * a * a / s
    out = {"dx": d * s * i, "dzi": d * x * s * i * (1 - i),
           "dzr": torch.nn.functional.softplus(lam) * dq * r * (1 - r),
           "dlambda": torch.sigmoid(lam) * (dq * r).sum((0, 1)), "dh0": a[0] * d[0]}
    return h, out


def _time_first(t):
    return t.double().transpose(0, 1).contiguous()


def _layer64(x, s, dh=None):
    """The layer with projections on [L][B][D] tensors: h and the gradients."""
    L, B, D = x.shape
    flat = x.reshape(-1, D)
    w = {n: s[n].double() for n in ("Wr", "Wi", "br", "bi", "lam")}
    z = [torch.addmm(w["b" + k], flat, w["W" + k].t()).reshape(L, B, D) for k in "ri"]
    h, g = _scan64(x, z[0], z[1], w["lam"], None if s["h0"] is None else s["h0"].double(), dh)
    if g is None:
        return h, None
    out = {k: g[k] for k in ("dlambda", "dh0")}
    dx = g["dx"].reshape(-1, D)
    for k in "ri":
        dz = g["dz" + k].reshape(-1, D)
        dx = torch.addmm(dx, dz, w["W" + k])
        out["dW" + k], out["db" + k] = dz.t().contiguous() @ flat, dz.sum(0)
    return h, {"dx": dx.reshape(L, B, D), **out}


def _dropout_scale(case, site, seed, shape):
    """0 or 1 / (1 - p) of each element: Philox4x64-10 words, 32 bits an element."""
    n = math.prod(shape)
    start = ((site << 64) - 1) % (1 << 256)  # numpy steps the counter before it draws
    counter = np.array([(start >> (64 * k)) & (2 ** 64 - 1) for k in range(4)], dtype=np.uint64)
    bits = np.random.Philox(counter=counter, key=np.array([seed, 1], dtype=np.uint64))
    words = bits.random_raw(-(-n // 8) * 4).view(np.uint32)[:n]
    p = np.float32(DROPOUT)
    keep = words >= np.uint32(int(np.floor(np.float64(p) * 2.0 ** 32)))
    return torch.from_numpy(keep).cuda().reshape(shape).double() / (1.0 - float(p))


def _model64(case, seed):
    flat, ids, targets = _model_inputs(case, seed)
    flat = flat.double().requires_grad_()
    p = {n: flat[o:o + math.prod(sh)].reshape(sh) for n, sh, o in _model_layout(case)[0]}
    B, T, D, ids, targets = case["B"], case["T"], case["D"], ids.long(), targets.long()
    norm = lambda v, g, b: torch.nn.functional.layer_norm(v, (D,), g, b, 1e-12)  # noqa: E731
    silu = torch.nn.functional.silu

    def drop(v, site):
        return v * _dropout_scale(case, site, seed, (B, T, D))

    H = norm(drop(p["emb"][ids] * (ids != 0).unsqueeze(-1), 0), p["emb_ln_g"], p["emb_ln_b"])
    for l in range(case["layers"]):
        q = lambda n: p["l%d.%s" % (l, n)]  # noqa: E731,B023
        hx, hz = H @ q("Wx").t() + q("bx"), H @ q("Wz").t() + q("bz")
        c = q("conv_b") + q("conv_w")[:, 0] * hx
        for j in range(1, min(TAPS, T)):
            c = c + q("conv_w")[:, j] * torch.nn.functional.pad(hx, (0, 0, j, 0))[:, :T]
        x = silu(c)
        _, i, a, s = _gates(x @ q("Wr").t() + q("br"), x @ q("Wi").t() + q("bi"), q("lambda"))
        h = _Recurrence.apply(a.transpose(0, 1).contiguous(),
                              (s * i * x).transpose(0, 1).contiguous()).transpose(0, 1)
        H = norm(H + drop((h * silu(hz)) @ q("Wo").t() + q("bo"), 1 + 2 * l), q("ln1_g"),
                 q("ln1_b"))
        H = norm(H + drop(silu(H @ q("W1").t() + q("b1")) @ q("W2").t() + q("b2"), 2 + 2 * l),
                 q("ln2_g"), q("ln2_b"))
    loss = torch.nn.functional.cross_entropy(H[:, -1] @ p["emb"].t(), targets)
    loss.backward()
    return {"loss": loss.detach().reshape(1), "grads": flat.grad}


def exact(case, seed):
    kind = case["kind"]
    if kind == "model":
        return _model64(case, seed)
    s = _inputs(case, seed)
    h0 = None if s["h0"] is None else s["h0"].double()
    back = lambda t: t.transpose(0, 1).contiguous()  # noqa: E731
    if kind == "step":
        h, _ = _layer64(s["x"].double()[None], {**s, "h0": s["h_prev"]})
        return {"h": h[0]}
    if kind == "scan":
        h, g = _scan64(*(_time_first(s[n]) for n in ("x", "zr", "zi")), s["lam"].double(), h0,
                       _time_first(s["dh"]))
        g = {k: back(v) if v.dim() == 3 else v for k, v in g.items()}
        return {"h": back(h), "hT": h[-1], **g}
    if kind == "layer":
        h, g = _layer64(_time_first(s["x"]), s, _time_first(s["dh"]))
        return {"h": back(h), "hT": h[-1], **g, "dx": back(g["dx"])}
    hx, hz = _time_first(s["hx"]), _time_first(s["hz"])
    cw, L = s["conv_w"].double(), hx.shape[0]
    c = s["conv_b"].double() + cw[:, 0] * hx
    for j in range(1, min(TAPS, L)):
        c[j:] += cw[:, j] * hx[:L - j]
    sc, sz = torch.sigmoid(c), torch.sigmoid(hz)
    if kind == "prefill":
        h, _ = _layer64(c * sc, s)
        return {"y": back(h * hz * sz), "hT": h[-1]}
    dy = _time_first(s["dy"])
    h, g = _layer64(c * sc, s, dy * hz * sz)
    dc = g.pop("dx") * sc * (1 + c * (1 - sc))
    dhx, dw = cw[:, 0] * dc, torch.zeros_like(cw)
    for j in range(min(TAPS, L)):
        if j:
            dhx[:L - j] += cw[:, j] * dc[j:]
        dw[:, j] = (dc[j:] * hx[:L - j]).sum((0, 1))
    if h0 is None:
        g.pop("dh0")
    return {"y": back(h * hz * sz), "h": back(h), "hT": h[-1], "dhx": back(dhx),
            "dhz": back(dy * h * sz * (1 + hz * (1 - sz))), "dconv_w": dw,
            "dconv_b": dc.sum((0, 1)), **g}
