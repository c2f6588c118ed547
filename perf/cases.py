"""Timed cases: what a user of the library has it evaluate, through the public Python entry points.

A case is one expression at one size: ``prepare`` draws the inputs on the GPU and derives the plan, ``run`` is one
pass (forward evaluation and every gradient, as one step of a program does it).  The expressions are the ones of
``workloads.py``; the sizes are its configurations, the benchmark's, and generic sizes around them.
"""
from __future__ import annotations

import math

import torch

from paper_1711_01348_amd import binding, workloads

DEVICE = "cuda"
DTYPE = {"f32": torch.float32, "f64": torch.float64}


# ------------------------------------------------------------------------------------------------
# the cases
# ------------------------------------------------------------------------------------------------

def listed():
    return [
        # the paper's worked expression at its printed size: a step of two calls on 2 KB of tensors, launches only
        dict(name="worked_8x6x5_f64", kind="worked", I=8, J=6, K=5, dtype="f64"),
        # the same expression at scale with a short sum: two large tensors streamed, a dense masked gradient
        dict(name="worked_8192x8192x5", kind="worked", I=8192, J=8192, K=5, dtype="f32"),
        # the sizes a program has when nobody rounds them: odd extents, rows of f that start anywhere
        dict(name="worked_3001x2047x7", kind="worked", I=3001, J=2047, K=7, dtype="f32"),
        # a long summed index: three contractions and their element-wise parts
        dict(name="worked_4096x4096x256", kind="worked", I=4096, J=4096, K=256, dtype="f32"),
        # index sum f_ij = exp(x_{i+j}): one gradient element per antidiagonal
        dict(name="index_sum_4096x4096", kind="index_sum", I=4096, J=4096, body="exp"),
        # strided 3 x 3 map with tanh: a convolution step whose tensors stay in the caches
        dict(name="strided_32x128x128", kind="strided", N=32, I=128, J=128, U=3, V=3, stride=2),
        # matrix product and its two gradients at the benchmark's size: the largest amount of work
        dict(name="matmul_4096_f32", kind="matmul", I=4096, J=4096, K=4096, dtype="f32", xt=False, yt=False),
        # a double precision product of ragged size (a solver's or a gradient check's)
        dict(name="matmul_1000x1203x777_f64", kind="matmul", I=1000, J=1203, K=777, dtype="f64", xt=False, yt=False),
        # dense layer tanh(b + x w), a user-written scalar program with an operand outside the sum
        dict(name="dense_512x1024x768", kind="dense", I=512, J=1024, K=768),
        # a user-written program with transcendental functions of every operand inside the sum
        dict(name="softplus_512x384x200", kind="softplus", I=512, J=384, K=200),
        # causal convolution over a long signal: a range of the sum that depends on the function index
        dict(name="causal_conv_262144x33", kind="conv", N=262144, K=33),
        # one gradient of the dense layer through its derived expressions (what second derivatives are built from)
        dict(name="derived_dense_512x512x512", kind="derived", I=512, J=512, K=512),
    ]


def _log(rng, lo, hi):
    """A size between lo and hi, spread over its logarithm; as often odd as not."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _bounded(rng, limits, product):
    """Sizes within their limits whose product stays below `product`."""
    while True:
        sizes = [_log(rng, lo, hi) for lo, hi in limits]
        if math.prod(sizes) <= product:
            return sizes


def draw(rng):
    kind = rng.choice(["worked", "worked", "worked_f64", "worked_long", "index_sum", "broadcast", "diagonal", "strided",
                       "matmul", "matmul", "matmul_f64", "dense", "dense", "softplus", "conv", "derived"])
    if kind == "worked":
        I, J = _bounded(rng, [(16, 8192), (16, 8192)], 8192 * 8192)
        return dict(kind="worked", I=I, J=J - J % 4 if rng.random() < 0.5 else J, K=rng.randint(1, 8), dtype="f32")
    if kind == "worked_f64":
        I, J, K = _bounded(rng, [(4, 1024), (4, 1024), (1, 16)], 1 << 22)
        return dict(kind="worked", I=I, J=J, K=K, dtype="f64")
    if kind == "worked_long":
        I, J = _bounded(rng, [(64, 4096), (64, 4096)], 4096 * 4096)
        return dict(kind="worked", I=I, J=max(64, J - J % 4), K=32 * rng.randint(1, 8), dtype="f32")
    if kind in ("index_sum", "broadcast"):
        I, J = _bounded(rng, [(16, 8192), (16, 8192)], 4096 * 4096)
        return dict(kind=kind, I=I, J=J - J % 4 if rng.random() < 0.5 else J,
                    body=rng.choice(["exp", "sq", "sin", "cube"]))
    if kind == "diagonal":
        return dict(kind=kind, I=_log(rng, 16, 8192), body=rng.choice(["exp", "sq", "sin", "cube"]))
    if kind == "strided":
        U, V = rng.choice([(3, 3), (3, 3), (2, 2), (5, 5), (1, 3), (7, 7)])
        # batches of a multiple of four images, of any size
        N, I, J = _bounded(rng, [(1, 16), (8, 256), (8, 256)], 32 * 128 * 128 // 2)
        return dict(kind="strided", N=4 * N, I=I, J=J, U=U, V=V, stride=rng.randint(1, 3))
    if kind == "matmul":
        I, J, K = _bounded(rng, [(32, 4096), (32, 4096), (32, 4096)], 1 << 33)
        if rng.random() < 0.7:
            I, J, K = (max(32, s - s % 4) for s in (I, J, K))
        return dict(kind="matmul", I=I, J=J, K=K, dtype="f32", xt=rng.random() < 0.3, yt=rng.random() < 0.3)
    if kind == "matmul_f64":
        I, J, K = _bounded(rng, [(16, 1536), (16, 1536), (16, 1536)], 1 << 30)
        return dict(kind="matmul", I=I, J=J, K=K, dtype="f64", xt=rng.random() < 0.3, yt=rng.random() < 0.3)
    if kind == "softplus":
        I, J, K = _bounded(rng, [(16, 1024), (16, 1024), (4, 512)], 1 << 26)
        return dict(kind="softplus", I=I, J=J, K=K)
    if kind == "conv":
        N, K = _bounded(rng, [(1 << 10, 1 << 20), (2, 128)], 1 << 25)
        return dict(kind="conv", N=N, K=K)
    I, J, K = _bounded(rng, [(16, 2048), (16, 2048), (16, 2048)], 1 << 29)
    return dict(kind=kind, I=I, J=J, K=K)


# ------------------------------------------------------------------------------------------------
# expressions and inputs
# ------------------------------------------------------------------------------------------------

def _expr(case):
    k = case["kind"]
    if k == "worked":
        return workloads.worked_expr(case["I"], case["J"], case["K"], case["dtype"])
    if k in ("index_sum", "broadcast", "diagonal"):
        e = (workloads.index_sum_exp_expr(case["I"], case["J"], "f32") if k == "index_sum" else
             workloads.broadcast_sq_expr(case["I"], case["J"], "f32") if k == "broadcast" else
             workloads.diagonal_sq_expr(case["I"], "f32"))
        e.body = case["body"] if "body" in case else e.body
        return e
    if k == "strided":
        return workloads.strided_tanh_expr(case["N"], case["I"], case["J"], case["U"], case["V"], case["stride"], "f32")
    if k == "matmul":
        return workloads.matmul_expr(case["I"], case["J"], case["K"], case["dtype"], case["xt"], case["yt"])
    if k in ("dense", "derived"):
        return workloads.dense_layer_expr(case["I"], case["J"], case["K"], "f32")
    if k == "softplus":
        return workloads.softplus_ratio_expr(case["I"], case["J"], case["K"], "f32")
    if k == "conv":
        return workloads.causal_convolution_expr(case["N"], case["K"], "f32")
    raise ValueError(k)


def _ranges(case):
    """Uniform range of every argument tensor, those of workloads.py."""
    k = case["kind"]
    if k == "worked":
        # c scales with 1 / K and d shrinks for a long sum, so that f stays of order one
        return [(-1, 1), (-1, 1), (0, 1.0 / case["K"]), (-0.5, 0.5) if case["K"] <= 16 else (-0.2, 0.2)]
    if k == "strided":
        return [(-1, 1), (-0.5, 0.5)]
    if k in ("dense", "derived"):
        h = math.sqrt(3.0 / case["K"])      # pre-activations of order one
        return [(-1, 1), (-h, h), (-0.5, 0.5)]
    return [(-1, 1)] * 3


def _inputs(case, seed):
    e = _expr(case)
    dt = DTYPE[e.dtype]
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)

    def uniform(shape, lo, hi):
        return torch.rand(tuple(shape), generator=gen, dtype=dt, device=DEVICE).mul_(hi - lo).add_(lo)

    args = [uniform(a.shape, *r) for a, r in zip(e.args, _ranges(case))]
    df = uniform(e.f_shape, -1, 1)
    return e, args, df


def prepare(case, seed):
    e, args, df = _inputs(case, seed)
    plan = binding.Plan(e)
    state = dict(args=args, df=df, plan=plan)
    if case["kind"] == "derived":
        grad = binding.DerivedGradient(plan, 0)
        state.update(derived=grad, dx=torch.empty_like(args[0]),
                     ws=torch.empty(max(grad.workspace_bytes, 1), dtype=torch.uint8, device=DEVICE))
        return state
    state.update(f=torch.empty_like(df), grads=[torch.empty_like(a) for a in args], ws=plan.workspace(DEVICE))
    return state


def run(state):
    args, df, ws = state["args"], state["df"], state["ws"]
    if "derived" in state:
        return [state["derived"].evaluate(args, df, out=state["dx"], ws=ws)]
    f = state["plan"].forward(args, out=state["f"], ws=ws)
    return [f] + state["plan"].backward(args, f, df, out=state["grads"], ws=ws)


# ------------------------------------------------------------------------------------------------
# what a pass cannot do without
# ------------------------------------------------------------------------------------------------

def work(case):
    e = _expr(case)
    size = 8 if e.dtype == "f64" else 4
    n_f = math.prod(e.f_shape)
    sizes = [math.prod(a.shape) for a in e.args]
    terms = n_f * math.prod(hi - lo + 1 for lo, hi in e.sums)
    k = case["kind"]
    read = list(sizes)
    if k == "worked":
        read[2] = case["I"]                 # only the diagonal of c is read; its gradient is dense
    elif k == "diagonal":
        read[0] = case["I"]
    if k == "derived":
        # x w for the seed and g w^T; x, w, b, df in, dx out
        return dict(bytes=size * (sum(read) + n_f + sizes[0]), flops=4 * terms)
    per_term = dict(worked=6, strided=6, matmul=6, dense=6, softplus=8, conv=6).get(k, 0)
    if k == "softplus":
        per_function = 4
    else:
        per_function = 3
    return dict(bytes=size * (sum(read) + 2 * n_f + sum(sizes)), flops=per_term * terms + per_function * n_f)


# ------------------------------------------------------------------------------------------------
# tolerance and the values themselves in 64 bits
# ------------------------------------------------------------------------------------------------

def tolerance(case):
    """About four times the error against exact() that was measured over the listed and sixty drawn cases."""
    if case.get("dtype") == "f64":
        return {"rel": 1e-14, "max": 2e-13}
    if case["kind"] == "matmul":        # sums of up to 4096 products in 32 bits
        return {"rel": 5e-6, "max": 4e-5}
    if case["kind"] == "worked":        # the gradient of c is almost all zeros: its largest error over its rms
        return {"rel": 1.2e-6, "max": 1e-4}
    return {"rel": 6e-7, "max": 4e-6}


def _phi(body, x):
    """phi(x) and phi'(x)."""
    if body == "sq":
        return x * x, 2 * x
    if body == "cube":
        return x ** 3, 3 * x * x
    if body == "sin":
        return torch.sin(x), torch.cos(x)
    return torch.exp(x), torch.exp(x)


def _antidiagonal_sums(v):
    """out[m] = sum of v[i, m - i]."""
    I, J = v.shape
    pad = torch.zeros(I, I + J, dtype=v.dtype, device=v.device)
    pad[:, :J] = v
    return pad.reshape(-1)[:I * (I + J - 1)].reshape(I, I + J - 1).sum(0)


def exact(case, seed):
    _, args, df = _inputs(case, seed)
    args, df = [a.double() for a in args], df.double()
    k = case["kind"]
    if k == "worked":
        return _exact_worked(case, args, df)
    if k in ("index_sum", "broadcast", "diagonal"):
        x, = args
        if k == "diagonal":
            f, d = _phi(case["body"], x.diagonal())
            return [f, torch.diag(df * d)]
        f, d = _phi(case["body"], x)
        if k == "broadcast":
            return [f[:, None].expand(case["I"], case["J"]).contiguous(), df.sum(1) * d]
        return [f.unfold(0, case["J"], 1).contiguous(), _antidiagonal_sums(df) * d]
    if k == "strided":
        x, w = args
        s, I, J = case["stride"], case["I"], case["J"]
        taps = [(u, v) for u in range(case["U"]) for v in range(case["V"])]

        def window(t, u, v):
            return t[:, u:u + s * (I - 1) + 1:s, v:v + s * (J - 1) + 1:s]

        acc = torch.zeros_like(df)
        for u, v in taps:
            acc += window(x, u, v) * w[u, v]
        f = torch.tanh(acc)
        t = df * (1 - f * f)
        dx, dw = torch.zeros_like(x), torch.zeros_like(w)
        for u, v in taps:
            window(dx, u, v).add_(t * w[u, v])
            dw[u, v] = (t * window(x, u, v)).sum()
        return [f, dx, dw]
    if k == "matmul":
        x, y = args
        X, Y = (x.t() if case["xt"] else x), (y.t() if case["yt"] else y)
        dX, dY = df @ Y.t(), X.t() @ df
        return [X @ Y, dX.t().contiguous() if case["xt"] else dX, dY.t().contiguous() if case["yt"] else dY]
    if k in ("dense", "derived"):
        x, w, b = args
        f = torch.tanh(x @ w + b)
        g = df * (1 - f * f)
        if k == "derived":
            return [g @ w.t()]
        return [f, g @ w.t(), x.t() @ g, g.sum(0)]
    if k == "softplus":
        x, y, z = args
        zk = z.unfold(0, case["K"], 1)                       # z_{i+k}
        den, ex, ry = 2 + torch.cos(zk), torch.exp(x), torch.sqrt(y * y + 1)
        A = ex / den
        s = A @ ry
        g = df / (1 + s)
        gy = g @ ry.t()
        return [torch.log1p(s), A * gy, (A.t() @ g) * (y / ry),
                _antidiagonal_sums(A * gy * torch.sin(zk) / den)]
    if k == "conv":
        x, w = args
        N = case["N"]
        f, dx, dw = torch.zeros_like(df), torch.zeros_like(x), torch.zeros_like(w)
        for q in range(case["K"]):
            f[q:] += x[:N - q] * w[q]
            dx[:N - q] += df[q:] * w[q]
            dw[q] = (df[q:] * x[:N - q]).sum()
        return [f, dx, dw]
    raise ValueError(k)


def _exact_worked(case, args, df):
    a, b, c, d = args
    I, K = case["I"], case["K"]
    ci = c.diagonal()
    D = (d ** 3).unfold(0, K, 1)[:I].sum(1)
    na, nb = (a * a).sum(1), (b * b).sum(1)
    f = torch.exp(-(ci[:, None] * (na[:, None] + nb[None, :] + 2 * (a @ b.t())) + D[:, None]))
    g = df * f
    r, P = g.sum(1), g @ b
    da = -2 * ci[:, None] * (a * r[:, None] + P)
    cg = ci[:, None] * g
    db = -2 * (cg.t() @ a + b * cg.sum(0)[:, None])
    dc = torch.zeros_like(c)
    dc.diagonal().copy_(-(na * r + 2 * (a * P).sum(1) + g @ nb))
    dd = torch.zeros_like(d)
    for q in range(K):
        dd[q:q + I] += r
    return [f, da, db, dc, -3 * d * d * dd]
