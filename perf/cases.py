"""Performance cases of the 3D-DSA library: what its users run, through its public calls.

A case is one pass of a program that holds its inputs on the GPU: "forward" is an inference
call (no LSE, no residual), "step" a training step of one layer (the forward and the backward
with every output and gradient).  Four operators: `dsa` (3D deformable slide attention), `pw`
(its predicted-weights variant), `conv` (the depthwise 3D convolution of Eq. (1) and of the
offset network) and `win` (the shifted-window baseline).  Grids, heads, kernels and value
distributions are those of the repository's workloads, on fewer frames where a whole clip would
only repeat the work.
"""
import math

import torch

import paper_2607_22696_amd as dsa


def _attention(op, name, kind, grid, heads, head_dim, kernel, dtype, offsets, batch=1):
    T, H, W = grid
    return {"name": name, "op": op, "pass": kind, "B": batch, "T": T, "H": H, "W": W,
            "heads": heads, "head_dim": head_dim, "kt": kernel[0], "kh": kernel[1],
            "kw": kernel[2], "dtype": dtype, "offsets": offsets}


def _conv(name, kind, grid, channels, kernel, dtype, batch=1):
    T, H, W = grid
    return {"name": name, "op": "conv", "pass": kind, "B": batch, "T": T, "H": H, "W": W,
            "channels": channels, "kt": kernel[0], "kh": kernel[1], "kw": kernel[2],
            "dtype": dtype}


def _window(name, kind, grid, heads, head_dim, window, shift, batch=1):
    T, H, W = grid
    return {"name": name, "op": "win", "pass": kind, "B": batch, "T": T, "H": H, "W": W,
            "heads": heads, "head_dim": head_dim, "wt": window[0], "wh": window[1],
            "ww": window[2], "st": shift[0], "sh": shift[1], "sw": shift[2], "dtype": "bf16"}


def listed():
    return [
        # the smallest call: a unit-test-sized grid, where launches and host work are the time
        _attention("dsa", "dsa_step_4x8x8_f32", "step", (4, 8, 8), 2, 32, (3, 3, 3), "f32",
                   "normal0.5"),
        # inference on a short low-resolution clip (16,384 tokens)
        _attention("dsa", "dsa_fwd_16x32x32", "forward", (16, 32, 32), 8, 64, (3, 3, 3), "bf16",
                   "uniform2"),
        # an ordinary training step: 64 frames of a 34 x 60 latent grid
        _attention("dsa", "dsa_step_64x34x60", "step", (64, 34, 60), 16, 64, (3, 3, 3), "bf16",
                   "uniform2"),
        # inference at the 1080p latent resolution, 522,240 tokens, 24 heads x 128
        _attention("dsa", "dsa_fwd_64x68x120", "forward", (64, 68, 120), 24, 128, (3, 3, 3),
                   "bf16", "normal1"),
        # training with a larger neighbourhood and fast motion (offsets of up to 8 tokens)
        _attention("dsa", "dsa_step_3x5x5_wide", "step", (32, 34, 60), 24, 128, (3, 5, 5), "bf16",
                   "uniform8"),
        # training with the paper's 3 x 7 x 7 neighbourhood
        _attention("dsa", "dsa_step_3x7x7", "step", (16, 34, 60), 24, 128, (3, 7, 7), "bf16",
                   "normal1"),
        # training in fp32 on an odd grid with two clips in the batch
        _attention("dsa", "dsa_step_9x33x47_f32", "step", (9, 33, 47), 6, 64, (3, 3, 3), "f32",
                   "normal1", batch=2),
        # the predicted-weights variant's training step on the ordinary grid
        _attention("pw", "pw_step_64x34x60", "step", (64, 34, 60), 16, 64, (3, 3, 3), "bf16",
                   "uniform2"),
        # the convolution term of Eq. (1) beside a 1080p attention layer, training
        _conv("conv_step_64x68x120", "step", (64, 68, 120), 3072, (3, 3, 3), "bf16"),
        # the offset network's depthwise layer trained in fp32
        _conv("conv_step_16x34x60_f32", "step", (16, 34, 60), 1024, (3, 3, 3), "f32"),
        # the window baseline: inference on the ordinary grid, plain windows
        _window("win_fwd_64x34x60", "forward", (64, 34, 60), 16, 64, (3, 16, 16), (0, 0, 0)),
        # the window baseline at the 1080p resolution: training, shifted windows
        _window("win_step_32x68x120", "step", (32, 68, 120), 24, 128, (3, 16, 16), (1, 8, 8)),
    ]


# ----------------------------------------------------------------------------- drawn cases

_POINT_CHANNELS = 32 * 34 * 60 * 24 * 75 * 128      # dsa_step_3x5x5_wide
_CONV_TAPS = 64 * 68 * 120 * 3072 * 27              # conv_step_64x68x120
_WINDOW_PRODUCTS = 32 * 68 * 120 * 24 * 768 * 128   # win_step_32x68x120


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _grid(rng):
    return _log_int(rng, 2, 64), _log_int(rng, 6, 68), _log_int(rng, 6, 120)


def _halve(case, cost, limit):
    """The case with its largest grid side halved until it costs at most `limit`."""
    while cost(case) > limit:
        side = max(("T", "H", "W"), key=lambda a: case[a])
        case[side] = max(1, case[side] // 2)
    return case


def draw(rng):
    op = rng.choice(("dsa", "dsa", "dsa", "pw", "conv", "win"))
    kind = rng.choice(("forward", "step", "step"))
    batch = rng.choice((1, 1, 2))
    if op in ("dsa", "pw"):
        case = _attention(op, "", kind, _grid(rng), rng.choice((1, 2, 3, 6, 8, 12, 16, 24)),
                          rng.choice((32, 64, 64, 128, 128)),
                          rng.choice(((1, 3, 3), (3, 3, 3), (3, 3, 3), (3, 5, 5), (3, 7, 7))),
                          rng.choice(("bf16", "bf16", "bf16", "f32")),
                          rng.choice(("normal0.5", "normal1", "uniform2", "uniform8")), batch)
        case = _halve(case, lambda c: c["B"] * c["T"] * c["H"] * c["W"] * c["heads"] * c["kt"] *
                      c["kh"] * c["kw"] * c["head_dim"] * (2 if c["dtype"] == "f32" else 1),
                      _POINT_CHANNELS)
    elif op == "conv":
        case = _conv("", kind, _grid(rng), 2 * _log_int(rng, 16, 1536),
                     rng.choice(((3, 3, 3), (3, 3, 3), (1, 3, 3), (3, 5, 5), (1, 7, 7))),
                     rng.choice(("bf16", "bf16", "f32")), batch)
        case = _halve(case, lambda c: c["B"] * c["T"] * c["H"] * c["W"] * c["channels"] *
                      c["kt"] * c["kh"] * c["kw"] * (2 if c["dtype"] == "f32" else 1),
                      _CONV_TAPS)
    else:
        window = rng.choice(((3, 16, 16), (3, 16, 16), (3, 8, 8), (8, 7, 7), (4, 16, 16)))
        shift = tuple(w // 2 for w in window) if rng.random() < 0.5 else (0, 0, 0)
        case = _window("", kind, _grid(rng), rng.choice((1, 3, 6, 8, 12, 16, 24)),
                       rng.choice((64, 128)), window, shift, batch)
        case = _halve(case, lambda c: c["B"] * c["T"] * c["H"] * c["W"] * c["heads"] *
                      c["wt"] * c["wh"] * c["ww"] * c["head_dim"], _WINDOW_PRODUCTS)
    del case["name"]
    return case


# ----------------------------------------------------------------------------- inputs and pass

_DTYPE = {"bf16": torch.bfloat16, "f32": torch.float32}


def _normal(gen, shape, std=1.0, dtype=torch.float32):
    return torch.randn(shape, generator=gen, device="cuda").mul_(std).to(dtype)


def _offsets(gen, shape, law):
    """Learned offsets: small after a zero-initialised offset network, about one token in
    ordinary motion, up to 8 tokens in fast motion."""
    if law.startswith("uniform"):
        a = float(law[7:])
        return torch.rand(shape, generator=gen, device="cuda").mul_(2 * a).sub_(a)
    return _normal(gen, shape, float(law[6:])).clamp_(-3.0, 3.0)


def _kernel(case):
    return case["kt"], case["kh"], case["kw"]


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    dt = _DTYPE[case["dtype"]]
    grid = (case["B"], case["T"], case["H"], case["W"])
    step = case["pass"] == "step"
    s = {"op": case["op"], "step": step}
    if case["op"] == "conv":
        C, taps = case["channels"], case["kt"] * case["kh"] * case["kw"]
        s["x"] = _normal(gen, grid + (C,), dtype=dt)
        s["weight"] = _normal(gen, (C,) + _kernel(case), taps ** -0.5)
        s["bias"] = _normal(gen, (C,), 0.1)
        if step:
            s["dy"] = _normal(gen, grid + (C,), dtype=dt)
        return s
    rows = grid + (case["heads"],)
    names = ["v"] if case["op"] == "pw" else ["q", "k", "v"]
    for name in names + (["dout"] if step else []):
        s[name] = _normal(gen, rows + (case["head_dim"],), dtype=dt)
    if case["op"] == "win":
        s["geometry"] = {"window": (case["wt"], case["wh"], case["ww"]),
                         "shift": (case["st"], case["sh"], case["sw"])}
        return s
    P = case["kt"] * case["kh"] * case["kw"]
    s["offsets"] = _offsets(gen, rows + (P, 3), case["offsets"])
    if case["op"] == "pw":
        s["logits"] = _normal(gen, rows + (P,), 1.5)
    s["geometry"] = {"kernel": _kernel(case)}
    return s


def run(state):
    s, step = state, state["step"]
    if s["op"] == "dsa":
        out, lse = dsa.forward(s["q"], s["k"], s["v"], s["offsets"], need_lse=step,
                               **s["geometry"])
        if not step:
            return {"out": out}
        dq, dk, dv, doff = dsa.backward(s["q"], s["k"], s["v"], s["offsets"], lse, s["dout"],
                                        **s["geometry"])
        return {"out": out, "lse": lse, "dq": dq, "dk": dk, "dv": dv, "d_offsets": doff}
    if s["op"] == "pw":
        out, lse = dsa.pw_forward(s["logits"], s["v"], s["offsets"], need_lse=step,
                                  **s["geometry"])
        if not step:
            return {"out": out}
        dlogits, dv, doff = dsa.pw_backward(s["logits"], s["v"], s["offsets"], lse, s["dout"],
                                            **s["geometry"])
        return {"out": out, "lse": lse, "dlogits": dlogits, "dv": dv, "d_offsets": doff}
    if s["op"] == "conv":
        y = dsa.dwconv3d_forward(s["x"], s["weight"], s["bias"])
        if not step:
            return {"y": y}
        dx, dw, db = dsa.dwconv3d_backward(s["x"], s["weight"], s["dy"])
        return {"y": y, "dx": dx, "dweight": dw, "dbias": db}
    out, lse, res = dsa.win_forward(s["q"], s["k"], s["v"], need_lse=step, need_residual=step,
                                    **s["geometry"])
    if not step:
        return {"out": out}
    dq, dk, dv = dsa.win_backward(s["q"], s["k"], s["v"], out, res, lse, s["dout"],
                                  **s["geometry"])
    # out + res is the forward's result; the residual alone is rounding, not a result
    return {"out": out, "lse": lse, "dq": dq, "dk": dk, "dv": dv}


# ----------------------------------------------------------------------------- work

def _cuts(size, window, shift):
    """Intervals of one axis: cut at shift + n window and at the grid's ends."""
    cuts = sorted({0, size} | set(range(shift, size, window)))
    return list(zip(cuts[:-1], cuts[1:]))


def work(case):
    es = 2 if case["dtype"] == "bf16" else 4
    step = case["pass"] == "step"
    tokens = case["B"] * case["T"] * case["H"] * case["W"]
    if case["op"] == "conv":
        n, taps = tokens * case["channels"], case["kt"] * case["kh"] * case["kw"]
        small = case["channels"] * (taps + 1) * 4
        # x in, y out; dy in, fp32 dx out
        return {"bytes": n * (2 * es + (es + 4 if step else 0)) + small * (2 if step else 1),
                "flops": 2 * n * taps * (3 if step else 1)}
    rows, D = tokens * case["heads"], case["head_dim"]
    if case["op"] == "win":
        pairs = 1
        for size, w, s in ((case["T"], case["wt"], case["st"]), (case["H"], case["wh"], case["sh"]),
                           (case["W"], case["ww"], case["sw"])):
            pairs *= sum((b - a) ** 2 for a, b in _cuts(size, w, s))
        pairs *= case["B"] * case["heads"]
        # q, k, v in, out out; dout in, three fp32 gradients and the LSE out
        return {"bytes": rows * D * (4 * es + (es + 12 if step else 0)) + (rows * 4 if step else 0),
                "flops": pairs * D * (14 if step else 4)}
    P = case["kt"] * case["kh"] * case["kw"]
    if case["op"] == "pw":
        # v, offsets, logits in, out out; dout in, dv, d_offsets, dlogits and the LSE out
        return {"bytes": rows * (D * 2 * es + P * 16) +
                (rows * (D * (es + 4) + P * 16 + 4) if step else 0),
                "flops": rows * P * D * (48 if step else 16)}
    # q, k, v, offsets in, out out; dout in, three gradients, d_offsets and the LSE out
    return {"bytes": rows * (D * 4 * es + P * 12) +
            (rows * (D * (es + 12) + P * 12 + 4) if step else 0),
            "flops": rows * P * D * (112 if step else 32)}


def tolerance(case):
    # Four times the largest distance from `exact` that was measured.  bf16: the rounding of the
    # output itself (1.7e-3; the largest is half a unit in the last place, 3.9e-3).  fp32: the
    # sums of the whole path (5.2e-7).
    if case["dtype"] == "bf16":
        return {"rel": 7e-3, "max": 2e-2}
    return {"rel": 2e-6, "max": 1e-4}


# ----------------------------------------------------------------------------- 64-bit results

_CHUNK = 1 << 26  # fp64 values of one gathered block of corner rows


def _corners(case, off, tok):
    """Corner rows (N for a corner outside the grid), weights and their position derivatives of
    the points of tokens `tok`: [n, P, 8] each, the derivatives with a last axis (x, y, z).
    The position is formed in fp32, as the operator defines it."""
    T, H, W = case["T"], case["H"], case["W"]
    kt, kh, kw = _kernel(case)
    p = torch.arange(kt * kh * kw, device=tok.device)
    base = ((tok % W)[:, None] + p % kw - (kw - 1) // 2,
            (tok // W % H)[:, None] + p // kw % kh - (kh - 1) // 2,
            (tok // (H * W))[:, None] + p // (kw * kh) - (kt - 1) // 2)
    low, frac = [], []
    for a, size in enumerate((W, H, T)):
        pos = (base[a].float() + off[..., a]).clamp(-2.0, size + 1.0).double()
        low.append(pos.floor())
        frac.append(pos - low[-1])
    rows, weights, derivs = [], [], []
    for c in range(8):
        bit = (c & 1, c >> 1 & 1, c >> 2)
        at = [low[a].long() + bit[a] for a in range(3)]
        w = [frac[a] if bit[a] else 1.0 - frac[a] for a in range(3)]
        sign = [1.0 if b else -1.0 for b in bit]
        ok = (at[0] >= 0) & (at[0] < W) & (at[1] >= 0) & (at[1] < H) & (at[2] >= 0) & (at[2] < T)
        rows.append(torch.where(ok, (at[2] * H + at[1]) * W + at[0], T * H * W))
        weights.append(w[0] * w[1] * w[2])
        derivs.append(torch.stack([sign[0] * w[1] * w[2], sign[1] * w[0] * w[2],
                                   sign[2] * w[0] * w[1]], -1))
    return torch.stack(rows, 2), torch.stack(weights, 2), torch.stack(derivs, 2)


def _exact_attention(case, s):
    B, N, heads = case["B"], case["T"] * case["H"] * case["W"], case["heads"]
    D, P = case["head_dim"], case["kt"] * case["kh"] * case["kw"]
    step, pw = s["step"], case["op"] == "pw"
    rows = B * N * heads
    if rows * P * D > (1 if step else 3) * _POINT_CHANNELS or (step and 4.0 * N * rows * D > 1e14):
        return None
    scale = D ** -0.5

    def flat(x):
        return x.reshape((B, N, heads) + tuple(x.shape[5:]))

    t = {n: flat(s[n]) for n in ("q", "k", "v", "dout", "offsets", "logits") if n in s}
    f64 = dict(dtype=torch.float64, device="cuda")
    r = {"out": torch.empty((B, N, heads, D), **f64), "lse": torch.empty((B, N, heads), **f64),
         "dv": torch.zeros((B, N, heads, D), **f64) if step else None,
         "d_offsets": torch.empty((B, N, heads, P, 3), **f64) if step else None}
    if pw:
        r["dlogits"] = torch.empty((B, N, heads, P), **f64) if step else None
    else:
        r["dq"] = torch.empty((B, N, heads, D), **f64) if step else None
        r["dk"] = torch.zeros((B, N, heads, D), **f64) if step else None
    size = max(1, min(_CHUNK // (P * 8 * D), _CHUNK // N if step else N))
    for b in range(B):
        for m in range(heads):
            padded = {n: torch.cat([t[n][b, :, m].double(), torch.zeros((1, D), **f64)])
                      for n in ("k", "v") if n in t}
            for n0 in range(0, N, size):
                tok = torch.arange(n0, min(n0 + size, N), device="cuda")
                at = (b, slice(n0, n0 + len(tok)), m)
                idx, w, dw = _corners(case, t["offsets"][at], tok)
                vc = padded["v"][idx]
                if pw:
                    logit, qk, kc = t["logits"][at].double(), None, None
                else:
                    q = t["q"][at].double()
                    kc = padded["k"][idx]
                    qk = (kc * q[:, None, None]).sum(-1)
                    logit = scale * (w * qk).sum(-1)
                lse = torch.logsumexp(logit, -1)
                alpha = (logit - lse[:, None]).exp()
                r["lse"][at] = lse
                aw = alpha[..., None] * w
                r["out"][at] = (vc * aw[..., None]).sum((1, 2))
                if not step:
                    continue
                g = t["dout"][at].double()
                gv = (vc * g[:, None, None]).sum(-1)
                da = (w * gv).sum(-1)
                ds = alpha * (da - (alpha * da).sum(-1, keepdim=True))
                slope = alpha[..., None] * gv
                if pw:
                    r["dlogits"][at] = ds
                else:
                    sw = scale * ds[..., None] * w
                    slope = slope + scale * ds[..., None] * qk
                    r["dq"][at] = (kc * sw[..., None]).sum((1, 2))
                r["d_offsets"][at] = (dw * slope[..., None]).sum(2)
                # dV and dK: the corner weights of the tokens as a dense [tokens, N] matrix
                for name, coef, row in (("dv", aw, g),) + (() if pw else (("dk", sw, q),)):
                    dense = torch.zeros((len(tok), N + 1), **f64)
                    dense.scatter_add_(1, idx.flatten(1), coef.flatten(1))
                    r[name][b, :, m] += dense[:, :N].t() @ row
    shape = (B, case["T"], case["H"], case["W"])
    r = {n: x.reshape(shape + tuple(x.shape[2:])) for n, x in r.items() if x is not None}
    return r if step else {"out": r["out"]}


def _exact_conv(case, s):
    B, T, H, W, C = s["x"].shape
    k = _kernel(case)
    taps = k[0] * k[1] * k[2]
    if B * T * H * W * C * taps > _CONV_TAPS:
        return None
    step, half = s["step"], [(a - 1) // 2 for a in k]
    pad = (0, 0, half[2], half[2], half[1], half[1], half[0], half[0])
    f64 = dict(dtype=torch.float64, device="cuda")
    r = {"y": torch.empty(s["x"].shape, **f64)}
    if step:
        r.update(dx=torch.empty(s["x"].shape, **f64), dweight=torch.empty((C,) + k, **f64),
                 dbias=torch.empty((C,), **f64))
    for c0 in range(0, C, 64):
        at = slice(c0, c0 + 64)
        w = s["weight"][at].double()
        x = torch.nn.functional.pad(s["x"][..., at].double(), pad)
        y = s["bias"][at].double().expand((B, T, H, W, -1)).clone()
        if step:
            dy = s["dy"][..., at].double()
            padded = torch.nn.functional.pad(dy, pad)
            dx = torch.zeros_like(dy)
            r["dbias"][at] = dy.sum((0, 1, 2, 3))
        for a in range(k[0]):
            for e in range(k[1]):
                for f in range(k[2]):
                    near = x[:, a:a + T, e:e + H, f:f + W]
                    y += near * w[:, a, e, f]
                    if step:
                        r["dweight"][at, a, e, f] = (near * dy).sum((0, 1, 2, 3))
                        dx += padded[:, k[0] - 1 - a:k[0] - 1 - a + T,
                                     k[1] - 1 - e:k[1] - 1 - e + H,
                                     k[2] - 1 - f:k[2] - 1 - f + W] * w[:, a, e, f]
        r["y"][..., at] = y
        if step:
            r["dx"][..., at] = dx
    return r


def _exact_window(case, s):
    B, T, H, W, heads, D = s["q"].shape
    step, scale = s["step"], D ** -0.5
    f64 = dict(dtype=torch.float64, device="cuda")
    r = {"out": torch.empty(s["q"].shape, **f64)}
    if step:
        r.update({n: torch.empty(s["q"].shape, **f64) for n in ("dq", "dk", "dv")})
        r["lse"] = torch.empty(s["q"].shape[:5], **f64)
    (wt, wh, ww), (st, sh, sw) = s["geometry"]["window"], s["geometry"]["shift"]
    for b in range(B):
        for t0, t1 in _cuts(T, wt, st):
            for i0, i1 in _cuts(H, wh, sh):
                for j0, j1 in _cuts(W, ww, sw):
                    at = (b, slice(t0, t1), slice(i0, i1), slice(j0, j1))

                    def box(x):  # [heads, tokens of the box, D]
                        return x[at].double().flatten(0, 2).transpose(0, 1).contiguous()

                    def put(name, x):
                        r[name][at] = x.transpose(0, 1).reshape(r[name][at].shape)

                    q, k, v = box(s["q"]), box(s["k"]), box(s["v"])
                    logit = scale * (q @ k.transpose(1, 2).contiguous())
                    lse = torch.logsumexp(logit, -1)
                    p = (logit - lse[..., None]).exp()
                    put("out", p @ v)
                    if not step:
                        continue
                    g = box(s["dout"])
                    dp = g @ v.transpose(1, 2).contiguous()
                    ds = scale * p * (dp - (p * dp).sum(-1, keepdim=True))
                    put("lse", lse)
                    put("dq", ds @ k)
                    put("dk", ds.transpose(1, 2).contiguous() @ q)
                    put("dv", p.transpose(1, 2).contiguous() @ g)
    return r


def exact(case, seed):
    s = prepare(case, seed)
    if case["op"] == "conv":
        return _exact_conv(case, s)
    if case["op"] == "win":
        return _exact_window(case, s)
    return _exact_attention(case, s)
