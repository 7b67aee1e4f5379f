"""What a program that uses this framework spends its GPU time on, as cases that can be timed.

  listed()             the cases, dicts of plain values
  draw(rng)            one more case of the same ranges
  prepare(case, seed)  what the program holds before the call: tables, batches, modules, inputs on the GPU
  run(state)           one pass through the public entry points; returns its outputs
  work(case)           bytes and operations one pass cannot do without
  exact(case, seed)    what run() returns, in 64-bit arithmetic and without the framework

Functions, domains, table sizes and point counts are those of the repository's
workloads: the Gaussian on [-5, 5] (normal points) or [-4, 4], the Lorentzian
on [-20, 20] and J0 on [0, 50] (uniform points), N = 16 .. 4096, up to 2^28
points, batches of up to 4096 tables of uneven size, and the per-pixel sums of
Gaussian kernels of the sample application (16 reference frames, 5 x 5 window).
"""

import math
import random

import numpy as np
import torch

import paper_1510_02975_amd as P

_FUNCS = {"gaussian": P.GAUSSIAN, "lorentzian": P.LORENTZIAN, "j0": P.BESSEL_J0}
_DOMAINS = {"gaussian": (-5.0, 5.0), "lorentzian": (-20.0, 20.0), "j0": (0.0, 50.0)}
_KDE_MODES = {"table": P.KDE_TABLE, "expf": P.KDE_EXPF, "fast_expf": P.KDE_FAST_EXPF}


def listed():
    return [
        # A thousand points through a small table: a scalar activation or one
        # request of a serving loop, where the call itself is the cost.
        dict(name="eval_1000", op="eval", f="gaussian", a=-4.0, b=4.0, N=64, optimal=False, proj=False,
             n=1000, shift=0),
        # The smallest of the paper's workloads: 2^20 points, N = 64 uniform.
        dict(name="eval_1m", op="eval", f="gaussian", a=-4.0, b=4.0, N=64, optimal=False, proj=False,
             n=1 << 20, shift=0),
        # A view that starts one element into an array (a chunk of a longer
        # signal), of an odd length.
        dict(name="eval_slice_12m", op="eval", f="lorentzian", a=-20.0, b=20.0, N=256, optimal=True, proj=True,
             n=12345679, shift=1),
        # The headline workload: 2^28 points, N = 1024 optimal projection.
        dict(name="eval_256m", op="eval", f="gaussian", a=-5.0, b=5.0, N=1024, optimal=True, proj=True,
             n=1 << 28, shift=0),
        # The largest table: high accuracy for an oscillating function.
        dict(name="eval_j0_n4096_128m", op="eval", f="j0", a=0.0, b=50.0, N=4096, optimal=True, proj=True,
             n=1 << 27, shift=0),
        # The gradient workload: y, dL/dx and dL/dv in one fused pass.
        dict(name="grad_64m", op="grad", f="gaussian", a=-5.0, b=5.0, N=512, optimal=True, proj=True,
             n=1 << 26, shift=0),
        # A trainable table inside a network: autograd forward and backward
        # over one activation of 128 x 1024.
        dict(name="train_131k", op="train", f="gaussian", a=-5.0, b=5.0, N=128, optimal=True, proj=True,
             n=128 * 1024, shift=0),
        # The function changes between calls: rebuild the table in place, then
        # evaluate a block of points with it.
        dict(name="retune_1m", op="retune", f="gaussian", a=-5.0, b=5.0, N=1024, optimal=True, proj=True,
             n=1 << 20, shift=0),
        # A small batch: 64 tables, a few hundred to a few thousand points each.
        dict(name="batch_64", op="batch", T=64, total=100003, layout=5),
        # The many-table workload: 4096 tables of uneven size, 2^28 points.
        dict(name="batch_4096", op="batch", T=4096, total=1 << 28, layout=2),
        # The same kind of batch trained: fused forward and backward.
        dict(name="batch_grad_512", op="batch_grad", T=512, total=1 << 25, layout=3),
        # The sample application at 1080p with the paper's choice of table.
        dict(name="kde_1080p", op="kde", H=1080, W=1920, T=16, r=2, mode="table", N=64, optimal=False, sigma=6.0),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["eval", "eval", "eval", "grad", "grad", "train", "retune", "batch", "batch_grad", "kde"])
    if op in ("batch", "batch_grad"):
        T = _log_uniform(rng, 16, 4096 if op == "batch" else 1024)
        total = _log_uniform(rng, 1 << 16, (1 << 28) if op == "batch" else (1 << 26))
        return dict(op=op, T=T, total=max(total, 64 * T), layout=rng.randrange(1 << 20))
    if op == "kde":
        W = _log_uniform(rng, 176, 960)
        H = max(96, int(W * rng.choice([0.5625, 0.75, 0.8182])))
        return dict(op=op, H=H, W=W, T=rng.randint(4, 16), r=rng.choice([1, 2, 2]),
                    mode=rng.choice(["table", "table", "expf", "fast_expf"]), N=_log_uniform(rng, 32, 1024),
                    optimal=rng.random() < 0.5, sigma=rng.choice([4.0, 6.0, 10.0]))
    f = rng.choice(["gaussian", "gaussian", "lorentzian", "j0"])
    a, b = _DOMAINS[f]
    hi = {"eval": 1 << 28, "grad": 1 << 26, "train": 1 << 22, "retune": 1 << 24}[op]
    return dict(op=op, f=f, a=a, b=b, N=_log_uniform(rng, 16, 4096), optimal=rng.random() < 0.75,
                proj=rng.random() < 0.6, n=_log_uniform(rng, 1000, hi),
                shift=rng.choice([0, 0, 0, 1, 2, 3]) if op in ("eval", "grad") else 0)


# ---- inputs -----------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _points(case, gen):
    """case["n"] points, in an array that starts case["shift"] elements into its allocation."""
    n, shift = case["n"], case["shift"]
    base = torch.empty(n + shift, dtype=torch.float32, device="cuda")
    x = base[shift:]
    if case["f"] == "gaussian" and case["b"] == 5.0:
        # normal points; the forward workloads clip them to the domain, the gradient ones do not
        x.normal_(0.0, 1.0 if case["op"] in ("grad", "train") else 1.5, generator=gen)
        if case["op"] not in ("grad", "train"):
            x.clamp_(case["a"], case["b"])
    else:
        x.uniform_(case["a"], case["b"], generator=gen)
    return x


def _params(f, width=1.0):
    return (1.0,) if f == "j0" else (width, 1.0)


def _kinds(case):
    return (P.OPTIMAL if case["optimal"] else P.UNIFORM), (P.PROJ if case["proj"] else P.INTERP)


def _retune_widths(case, seed):
    """Two widths (or amplitudes) that a retuned table alternates between."""
    r = random.Random(int(seed))
    return r.uniform(0.6, 1.4), r.uniform(0.6, 1.4)


def _retune_params(f, w):
    return (w,) if f == "j0" else (w, 1.0)


def _batch_layout(case):
    """The tables of a batch and their point counts: a fixed draw per layout number."""
    r = random.Random(int(case["layout"]))
    specs, weights = [], []
    for _ in range(case["T"]):
        f = r.choice(["gaussian", "lorentzian", "j0"])
        w = math.exp(r.uniform(math.log(0.1), math.log(10.0)))
        a, b = _DOMAINS[f]
        if f != "j0":
            a, b = float(np.float32(a * w)), float(np.float32(b * w))
        specs.append(dict(f=f, params=_params(f, w), a=a, b=b,
                          N=int(round(math.exp(r.uniform(math.log(16.0), math.log(4096.0))))),
                          optimal=r.random() < 0.5, proj=r.random() < 0.5))
        weights.append(math.exp(r.uniform(math.log(2.0 ** 10), math.log(2.0 ** 20))))
    scale = case["total"] / sum(weights)
    counts = [max(1, int(w * scale)) for w in weights]
    offs = [0]
    for c in counts:
        offs.append(offs[-1] + c)
    return specs, counts, offs


def _batch_points(specs, counts, gen):
    n = torch.tensor(counts, device="cuda")
    lo = torch.tensor([s["a"] for s in specs], dtype=torch.float32, device="cuda")
    w = torch.tensor([s["b"] - s["a"] for s in specs], dtype=torch.float32, device="cuda")
    total = sum(counts)
    x = torch.rand(total, device="cuda", generator=gen)
    x.mul_(torch.repeat_interleave(w, n, output_size=total))
    return x.add_(torch.repeat_interleave(lo, n, output_size=total))


def _frames(case, gen):
    """A drifting colour field with sensor noise and a foreground square, RGBA8."""
    H, W, T = case["H"], case["W"], case["T"]
    yy = torch.arange(H, device="cuda", dtype=torch.float32)[:, None, None]
    xx = torch.arange(W, device="cuda", dtype=torch.float32)[None, :, None]
    phase = 6.2831853 * torch.rand(3, device="cuda", generator=gen)

    def scene(shift):
        v = 128.0 + 60.0 * torch.sin(0.02 * (xx + shift) + 0.03 * yy + phase)
        v = v + 4.0 * torch.randn((H, W, 3), device="cuda", generator=gen)
        return v

    def rgba(v):
        out = torch.full((H, W, 4), 255, dtype=torch.uint8, device="cuda")
        out[..., :3] = v.round().clamp(0, 255).to(torch.uint8)
        return out

    hist = torch.stack([rgba(scene(0.7 * t)) for t in range(T)])
    cur = scene(0.7 * T)
    s = max(4, min(H, W) // 6)
    cur[H // 3:H // 3 + s, W // 2:W // 2 + s] = 255.0 * torch.rand(3, device="cuda", generator=gen)
    return rgba(cur), hist


def _inputs(case, seed):
    gen = _gen(seed)
    op = case["op"]
    if op == "kde":
        return _frames(case, gen)
    if op in ("batch", "batch_grad"):
        specs, counts, _ = _batch_layout(case)
        x = _batch_points(specs, counts, gen)
    else:
        x = _points(case, gen)
    if op in ("grad", "train", "batch_grad"):
        return x, torch.randn(x.shape, device="cuda", generator=gen)
    return (x,)


# ---- a pass -----------------------------------------------------------------

def prepare(case, seed):
    op = case["op"]
    s = dict(case=dict(case), inputs=_inputs(case, seed))
    if op == "kde":
        s["table"] = P.pwl_build(P.GAUSSIAN, (1.0, 1.0), 0.0, 8.0, case["N"],
                                 P.OPTIMAL if case["optimal"] else P.UNIFORM, P.PROJ)
        return s
    if op in ("batch", "batch_grad"):
        specs, _, offs = _batch_layout(case)
        tabs = []
        for t in specs:
            part, vals = _kinds(t)
            tabs.append(P.pwl_build(_FUNCS[t["f"]], t["params"], t["a"], t["b"], t["N"], part, vals, check=False))
        s["batch"] = P.pwl_batch_create(tabs, offs)
        return s
    part, vals = _kinds(case)
    if op == "train":
        s["module"] = P.PWLTable(_FUNCS[case["f"]], _params(case["f"]), case["a"], case["b"], case["N"], part, vals)
        s["inputs"][0].requires_grad_(True)
        return s
    s["table"] = P.pwl_build(_FUNCS[case["f"]], _params(case["f"]), case["a"], case["b"], case["N"], part, vals)
    if op == "retune":
        s["widths"] = _retune_widths(case, seed)
        s["turn"] = 0
    return s


def run(s):
    case = s["case"]
    op = case["op"]
    if op == "eval":
        return P.pwl_eval(s["table"], s["inputs"][0])
    if op == "grad":
        return list(P.pwl_eval_backward(s["table"], *s["inputs"]))
    if op == "train":
        x, g = s["inputs"]
        m = s["module"]
        y = m(x)
        dx, dv = torch.autograd.grad(y, (x, m.values), g)
        return [y.detach(), dx, dv]
    if op == "retune":
        part, vals = _kinds(case)
        out = []
        for w in s["widths"]:
            P.pwl_rebuild(s["table"], _FUNCS[case["f"]], _retune_params(case["f"], w), case["a"], case["b"], part, vals)
            out.append(P.pwl_eval(s["table"], s["inputs"][0]))
        return out
    if op == "batch":
        return P.pwl_batch_eval(s["batch"], s["inputs"][0])
    if op == "batch_grad":
        return list(P.pwl_batch_eval_backward(s["batch"], *s["inputs"]))
    return P.pwl_kde(s["table"], _KDE_MODES[case["mode"]], s["inputs"][0], s["inputs"][1], case["r"],
                     (case["sigma"],) * 3)


def work(case):
    op = case["op"]
    if op == "kde":
        px = case["H"] * case["W"]
        taps = px * case["T"] * (2 * case["r"] + 1) ** 2
        # three differences, two products and one sum per tap
        return {"bytes": 4 * px * (case["T"] + 2), "flops": 6 * taps}
    if op in ("batch", "batch_grad"):
        specs, counts, _ = _batch_layout(case)
        n, tab = sum(counts), sum(8 * (t["N"] + 1) for t in specs)
        if op == "batch":
            return {"bytes": 8 * n + tab, "flops": 3 * n}
        return {"bytes": 16 * n + tab + tab // 2, "flops": 10 * n}
    n, tab = case["n"], 8 * (case["N"] + 1)
    if op == "eval":
        return {"bytes": 8 * n + tab, "flops": 3 * n}
    if op in ("grad", "train"):
        return {"bytes": 16 * n + tab + tab // 2, "flops": 10 * n}
    # two builds (256 N density samples of about 50 operations, optimal partition only) and evaluations
    return {"bytes": 12 * n + 2 * tab, "flops": 6 * n + (2 * 256 * 50 * case["N"] if case["optimal"] else 0)}


# ---- the same in 64 bits, without the framework -----------------------------

def _f64(f, p, x):
    if f == "gaussian":
        return p[1] * torch.exp(-(x * x) / (2.0 * p[0] * p[0]))
    if f == "lorentzian":
        return p[1] / (1.0 + (x / p[0]) ** 2)
    return p[0] * torch.special.bessel_j0(x)


def _f64_second(f, p, x):
    if f == "gaussian":
        s2 = p[0] * p[0]
        return p[1] * (x * x / (s2 * s2) - 1.0 / s2) * torch.exp(-(x * x) / (2.0 * s2))
    if f == "lorentzian":
        u2 = (x / p[0]) ** 2
        return p[1] * (6.0 * u2 - 2.0) / (p[0] * p[0] * (1.0 + u2) ** 3)
    z = torch.where(x == 0.0, torch.ones_like(x), x)
    return p[0] * torch.where(x == 0.0, torch.full_like(x, -0.5),
                              torch.special.bessel_j1(z) / z - torch.special.bessel_j0(z))


def _solve_tridiagonal(a, d, c, r):
    """Rows a[i] v[i-1] + d[i] v[i] + c[i] v[i+1] = r[i], diagonally dominant, by cyclic reduction."""
    n, s = d.numel(), 1

    def below(v, fill):
        return torch.cat([torch.full((min(s, n),), fill, dtype=v.dtype), v[:max(0, n - s)]])

    def above(v, fill):
        return torch.cat([v[s:], torch.full((min(s, n),), fill, dtype=v.dtype)])

    while s < n:
        al, ga = -a / below(d, 1.0), -c / above(d, 1.0)
        d, r, a, c = (d + al * below(c, 0.0) + ga * above(a, 0.0), r + al * below(r, 0.0) + ga * above(r, 0.0),
                      al * below(a, 0.0), ga * above(c, 0.0))
        s *= 2
    return r / d


def _table64(f, p, a, b, N, optimal, proj):
    """(knots, values) of a table: the knots rounded to FP32, as a table holds them, the values in 64 bits."""
    k = torch.arange(N + 1, dtype=torch.float64)
    X = a + (b - a) * k / N
    if optimal:
        M = 256 * N
        t = a + torch.arange(M + 1, dtype=torch.float64) * ((b - a) / M)
        d = torch.abs(_f64_second(f, p, t)) ** 0.4
        S = torch.cat([torch.zeros(1, dtype=torch.float64), torch.cumsum((d[1:] + d[:-1]) * ((b - a) / M / 2.0), 0)])
        tau = k[1:N] * (S[-1] / N)
        j = torch.searchsorted(S, tau).clamp(1, M)
        X[1:N] = t[j - 1] + (tau - S[j - 1]) / (S[j] - S[j - 1]) * ((b - a) / M)
        X[torch.abs(X) <= 1e-12 * (b - a)] = 0.0
    X[0], X[N] = a, b
    X = X.to(torch.float32).to(torch.float64)
    if not proj:
        return X, _f64(f, p, X)
    z, w = np.polynomial.legendre.leggauss(16)
    t, w = torch.from_numpy((1.0 + z) / 2.0), torch.from_numpy(w / 2.0)
    h = X[1:] - X[:-1]
    fq = _f64(f, p, X[:-1, None] + h[:, None] * t) * w
    zero = torch.zeros(1, dtype=torch.float64)
    rhs = torch.cat([h * (fq * (1.0 - t)).sum(1), zero]) + torch.cat([zero, h * (fq * t).sum(1)])
    hl, hr = torch.cat([zero, h]), torch.cat([h, zero])
    return X, _solve_tridiagonal(hl / 6.0, (hl + hr) / 3.0, hr / 6.0, rhs)


def _eval64(X, v, x, g=None):
    """y, and with g also dL/dx and dL/dv, of FP32 points on the GPU, in 64 bits."""
    X, v = X.cuda(), v.cuda()
    slope = (v[1:] - v[:-1]) / (X[1:] - X[:-1])
    n, step = x.numel(), 1 << 25
    y = torch.empty(n, dtype=torch.float64, device="cuda")
    dx = torch.empty_like(y) if g is not None else None
    dv = torch.zeros_like(X) if g is not None else None
    inner = X[1:-1].contiguous()
    for i in range(0, n, step):
        xs = x[i:i + step].double()
        xc = xs.clamp(X[0], X[-1])
        k = torch.searchsorted(inner, xc, right=True)
        d = xc - X[k]
        y[i:i + step] = v[k] + d * slope[k]
        if g is not None:
            gs = g[i:i + step].double()
            dx[i:i + step] = torch.where((xs >= X[0]) & (xs <= X[-1]), gs * slope[k], torch.zeros_like(gs))
            w = d / (X[k + 1] - X[k])
            dv += torch.bincount(k, (1.0 - w) * gs, minlength=X.numel())
            dv += torch.bincount(k + 1, w * gs, minlength=X.numel())
    return y if g is None else [y, dx, dv]


def exact(case, seed):
    op = case["op"]
    ins = [t.detach() for t in _inputs(case, seed)]
    if op == "kde":
        return _kde64(case, *ins)
    if op in ("batch", "batch_grad"):
        specs, _, offs = _batch_layout(case)
        parts = []
        for t, o0, o1 in zip(specs, offs[:-1], offs[1:]):
            X, v = _table64(t["f"], t["params"], t["a"], t["b"], t["N"], t["optimal"], t["proj"])
            parts.append(_eval64(X, v, *(u[o0:o1] for u in ins)))
        return torch.cat(parts) if op == "batch" else [torch.cat([q[k] for q in parts]) for k in range(3)]
    f = case["f"]
    args = (case["a"], case["b"], case["N"], case["optimal"], case["proj"])
    if op == "retune":
        return [_eval64(*_table64(f, _retune_params(f, w), *args), ins[0]) for w in _retune_widths(case, seed)]
    return _eval64(*_table64(f, _params(f), *args), *ins)


def _kde64(case, frame, hist):
    H, W, T, r = case["H"], case["W"], case["T"], case["r"]
    u = torch.arange(-255, 256, dtype=torch.float64) / case["sigma"]
    if case["mode"] == "table":
        X, v = _table64("gaussian", (1.0, 1.0), 0.0, 8.0, case["N"], case["optimal"], True)
        lut = _eval64(X, v, torch.abs(u).cuda())
    else:
        lut = torch.exp(-0.5 * u * u).cuda()
    f = frame[..., :3].long()
    out = torch.zeros((H, W), dtype=torch.float64, device="cuda")
    rows, cols = torch.arange(H, device="cuda"), torch.arange(W, device="cuda")
    for k in range(T):
        h = hist[k, ..., :3].long()
        for dy in range(-r, r + 1):
            hy = h[(rows + dy).clamp(0, H - 1)]
            for dx in range(-r, r + 1):
                d = f - hy[:, (cols + dx).clamp(0, W - 1)] + 255
                g = lut[d]
                out += g[..., 0] * g[..., 1] * g[..., 2]
    return out / (T * (2 * r + 1) ** 2)
