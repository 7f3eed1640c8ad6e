"""Shared helpers of the GPU parity tests: device transfer and the error metric.

Error metric (the tolerance the workloads state, "max relative error", read
with a floor so that it stays meaningful where h crosses zero): per output
tensor, err = max_i |g_i - o_i| / (|o_i| + rms(o)).  Bars: 1e-4 for fp32 I/O,
1e-2 for bf16 I/O with an fp32 state.
"""
import numpy as np

TOL = {"f32": 1e-4, "bf16": 1e-2}


def floored_rel_err(got, want):
    got = np.asarray(got, dtype=np.float64)
    want = np.asarray(want, dtype=np.float64)
    if want.size == 0:
        return 0.0
    rms = float(np.sqrt(np.mean(want * want)))
    denom = np.abs(want) + rms
    if rms == 0.0:
        return float(np.max(np.abs(got - want)))
    return float(np.max(np.abs(got - want) / denom))


def error_report(got, want):
    """Three views of the error of one output tensor: the floored relative
    error the bar applies to, the same with a floor of 1e-3 rms (close to a
    plain elementwise relative error wherever |want| is not tiny), and the
    normwise max|g - o| / max|o|."""
    got = np.asarray(got, dtype=np.float64)
    want = np.asarray(want, dtype=np.float64)
    if want.size == 0:
        return {"floored": 0.0, "tight": 0.0, "normwise": 0.0}
    diff = np.abs(got - want)
    rms = float(np.sqrt(np.mean(want * want)))
    mx = float(np.max(np.abs(want)))
    return {"floored": float(np.max(diff / (np.abs(want) + rms))) if rms else float(diff.max()),
            "tight": float(np.max(diff / (np.abs(want) + 1e-3 * rms))) if rms else float(diff.max()),
            "normwise": float(diff.max() / mx) if mx else float(diff.max())}


def report(tag, got, want):
    """Print the error report of one output (collected from the GPU logs)."""
    r = error_report(got, want)
    print(f"ERR {tag}: floored {r['floored']:.2e} tight {r['tight']:.2e} "
          f"normwise {r['normwise']:.2e}", flush=True)
    return r


def assert_close(got, want, io, name=""):
    err = floored_rel_err(got, want)
    assert np.all(np.isfinite(np.asarray(got, dtype=np.float64))), f"{name}: non-finite output"
    assert err <= TOL[io], f"{name}: floored relative error {err:.3e} > {TOL[io]:.0e}"
    return err


def dev(a, io="f32"):
    """numpy float32 array (bf16-representable when io == 'bf16') -> GPU tensor of the I/O dtype."""
    import torch
    t = torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32))
    if io == "bf16":
        t = t.to(torch.bfloat16)  # exact: the values are already bf16
    return t.cuda()


def dev32(a):
    import torch
    return None if a is None else torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()


def host(t):
    import torch
    return t.detach().to(torch.float32).cpu().numpy()


def gated_backward_from_h(hx, hz, conv_w, Wr, br, Wi, bi, lam, h, dy):
    """Gradients of the gated layer (zero initial state, no conv bias) in numpy's 64 bits, as
    the oracle's gated_backward but from a given h instead of one formed again: the
    reference of a backward that reads an h rounded to bf16."""
    hx, hz, conv_w, Wr, br, Wi, bi, lam, h, dy = (
        np.asarray(a, dtype=np.float64) for a in (hx, hz, conv_w, Wr, br, Wi, bi, lam, h, dy))
    B, L, D = hx.shape
    K = conv_w.shape[1]
    sig = lambda v: 1.0 / (1.0 + np.exp(-v))  # noqa: E731
    c = np.zeros_like(hx)
    for j in range(min(K, L)):
        c[:, j:] += conv_w[:, j] * hx[:, :L - j]
    sc, sz = sig(c), sig(hz)
    x = c * sc
    r, i = sig(x @ Wr.T + br), sig(x @ Wi.T + bi)
    sp = np.log1p(np.exp(lam))
    a, m = np.exp(-sp * r), np.sqrt(-np.expm1(-2.0 * sp * r))
    delta = dy * hz * sz
    for t in range(L - 2, -1, -1):
        delta[:, t] += a[:, t + 1] * delta[:, t + 1]
    hp = np.concatenate([np.zeros((B, 1, D)), h[:, :-1]], axis=1)
    dq = delta * (x * i * a * a / m - a * hp)
    dzr, dzi = sp * dq * r * (1 - r), delta * x * m * i * (1 - i)
    dc = (delta * m * i + dzr @ Wr + dzi @ Wi) * sc * (1 + c * (1 - sc))
    out = {"dhz": dy * h * sz * (1 + hz * (1 - sz)), "dlambda": sig(lam) * (dq * r).sum((0, 1)),
           "dhx": np.zeros_like(hx), "dconv_w": np.zeros_like(conv_w)}
    for j in range(min(K, L)):
        out["dhx"][:, :L - j] += conv_w[:, j] * dc[:, j:]
        out["dconv_w"][:, j] = (dc[:, j:] * hx[:, :L - j]).sum((0, 1))
    for k, dz in (("r", dzr), ("i", dzi)):
        out["dW" + k] = dz.reshape(-1, D).T @ x.reshape(-1, D)
        out["db" + k] = dz.sum((0, 1))
    return out
