"""Sums of products that separate over the function indices: run as dense products with 64-bit accumulation."""
import ctypes

import numpy as np
import pytest

import oracle
from paper_1711_01348_amd import check
from paper_1711_01348_amd import workloads as wl
from paper_1711_01348_amd.workloads import ArgSpec, ExprSpec


def grouped_expr(dtype):
    """f_abn = sum_kl x_abkl y_kln: two indices in every group."""
    a, b, n, k, l = 5, 7, 36, 3, 9
    unit = lambda *d: [[1 if c == q else 0 for c in range(5)] for q in d]
    return ExprSpec("mul", (a, b, n), [(0, k - 1), (0, l - 1)],
                    [ArgSpec("x", (a, b, k, l), unit(0, 1, 3, 4)), ArgSpec("y", (k, l, n), unit(3, 4, 2))], dtype)


def window_expr(dtype):
    """f_in = sum_k x_{2i+k} y_kn: an overlapping view of x; only the gradient of y is a dense product."""
    return ExprSpec("mul", (70, 33), [(0, 20)],
                    [ArgSpec("x", (160,), [[2, 0, 1]]), ArgSpec("y", (21, 33), [[0, 0, 1], [0, 1, 0]])], dtype)


def slack_expr(dtype):
    """y is larger than what is read of it: its gradient has zeros no product would write."""
    return ExprSpec("mul", (40, 37), [(0, 29)],
                    [ArgSpec("x", (40, 30), [[1, 0, 0], [0, 0, 1]]), ArgSpec("y", (33, 40), [[0, 0, 1], [0, 1, 0]])], dtype)


CASES = [(f"{I}x{J}x{K}_{dt}{'_xt' * xt}{'_yt' * yt}{'_swap' * sw}",
          lambda I=I, J=J, K=K, dt=dt, xt=xt, yt=yt, sw=sw: wl.matmul_expr(I, J, K, dt, xt, yt, sw))
         for I, J, K, xt, yt, sw in
         [(16, 16, 8, 0, 0, 0), (16, 17, 64, 0, 0, 1), (31, 33, 65, 0, 1, 0), (33, 65, 129, 1, 0, 0), (64, 97, 63, 1, 1, 1),
          (40, 23, 1100, 0, 0, 0), (130, 35, 513, 1, 1, 0), (257, 46, 70, 0, 1, 1),
          (16, 17, 2100, 0, 0, 0), (17, 33, 9000, 0, 1, 0)]
         for dt in ("f32", "f64")]
CASES += [(f"{make.__name__}_{dt}", lambda make=make, dt=dt: make(dt)) for make in (grouped_expr, window_expr, slack_expr)
          for dt in ("f32", "f64")]


def _run(plan, w, ws_bytes=None, skew=0, null=False):
    """Forward and backward through the C entry points with a workspace of ws_bytes (default: what the plan asks for), `skew` bytes
    off its alignment, or with a null pointer of that size."""
    import torch
    from paper_1711_01348_amd import binding as B
    args = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in w.arg_list()]
    df = torch.from_numpy(w.df).cuda()
    f = torch.full_like(df, float("nan"))
    grads = [torch.full_like(a, float("nan")) for a in args]
    ws = torch.empty(plan.workspace_bytes + 16, dtype=torch.uint8, device="cuda")
    n = plan.workspace_bytes if ws_bytes is None else ws_bytes
    ptrs = (ctypes.c_void_p * len(args))(*[t.data_ptr() for t in args])
    outs = (ctypes.c_void_p * len(args))(*[t.data_ptr() for t in grads])
    wp = ws.data_ptr() + skew if n and not null else None
    assert B.lib.tad_eval_forward(plan._h, ptrs, f.data_ptr(), wp, n, None) == 0
    assert B.lib.tad_eval_backward(plan._h, ptrs, f.data_ptr(), df.data_ptr(), outs, wp, n, None) == 0
    torch.cuda.synchronize()
    return f.cpu().numpy(), [g.cpu().numpy() for g in grads]


@pytest.mark.gpu
@pytest.mark.parametrize("name,make", CASES, ids=[c[0] for c in CASES])
def test_products_of_any_extents_and_orders(name, make):
    """Against the oracle; and with the workspace the general kernels need, which leaves the products out."""
    from paper_1711_01348_amd import binding as B
    expr = make()
    w = wl.random_inputs(expr, 77)
    plan, general = B.Plan(expr), B.Plan(expr, generic_only=True)
    f_ref, g_ref = oracle.forward(expr, w.arg_list()), oracle.backward(expr, w.arg_list(), w.df)
    for ws_bytes in (None, general.workspace_bytes):
        f, grads = _run(plan, w, ws_bytes)
        assert check.within(f, f_ref, expr.dtype), (name, ws_bytes, check.errors(f, f_ref))
        for g, r in zip(grads, g_ref):
            assert check.within(g, r, expr.dtype), (name, ws_bytes, check.errors(g, r))
            assert np.all(g[r == 0] == 0)


# products left to the kernels that store faster: of whole tiles in 32 bits (the sum, one gradient beside one that is a dense
# product, in either order), and forward sums of a few terms
SHORT = [(1300, 1300, 12, "f32", 0, 0), (1300, 1300, 12, "f32", 1, 1), (1300, 16, 1300, "f32", 0, 0), (20, 1300, 1200, "f32", 1, 0),
         (1300, 1300, 132, "f32", 0, 0), (65601, 17, 9, "f32", 0, 0), (16, 65537, 20, "f32", 0, 1), (1100, 1000, 9, "f64", 0, 0), (1100, 1000, 13, "f64", 0, 0)]


@pytest.mark.gpu
@pytest.mark.parametrize("I,J,K,dtype,xt,yt", SHORT)
def test_short_sums_on_either_side_of_the_line(I, J, K, dtype, xt, yt):
    from paper_1711_01348_amd import binding as B
    expr = wl.matmul_expr(I, J, K, dtype, xt, yt)
    w = wl.random_inputs(expr, 78)
    f, grads = _run(B.Plan(expr), w)
    assert check.within(f, oracle.forward(expr, w.arg_list()), dtype)
    for g, r in zip(grads, oracle.backward(expr, w.arg_list(), w.df)):
        assert check.within(g, r, dtype), check.errors(g, r)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_infinities_stay_in_their_rows_and_columns(dtype):
    """Edge tiles repeat rows and pad the sum: an infinity or a NaN in the last row, column or term reaches the results it
    belongs to and no others."""
    from paper_1711_01348_amd import binding as B
    I, J, K = 37, 41, 67
    expr = wl.matmul_expr(I, J, K, dtype)
    w = wl.random_inputs(expr, 5)
    x, y = w.arg_list()
    x[I - 1, K - 1] = np.inf
    y[K - 1, J - 1] = np.nan
    f, (dx, dy) = _run(B.Plan(expr), w)
    x64, y64, d64 = x.astype(np.float64), y.astype(np.float64), w.df.astype(np.float64)
    with np.errstate(invalid="ignore"):
        want = [(x64[:, :, None] * y64[None]).sum(1), (d64[:, None, :] * y64[None]).sum(2), (x64[:, :, None] * d64[:, None, :]).sum(0)]
    for got, ref in zip((f, dx, dy), want):
        assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isinf(got), np.isinf(ref))
        ok = np.isfinite(ref)
        assert check.within(np.where(ok, got, 0), np.where(ok, ref, 0), dtype)


@pytest.mark.gpu
@pytest.mark.parametrize("make", [lambda: wl.matmul_expr(40, 23, 1100, "f64"), lambda: wl.matmul_expr(37, 23, 1100, "f32"),
                                  lambda: wl.matmul_expr(40, 24, 30, "f64")], ids=["f64", "f32", "no_partial_sums"])
def test_no_partial_sums_where_there_is_no_workspace_for_them(make):
    """Partial sums are wanted, none of the family's kernels needs a workspace: a null pointer or one off its alignment gives
    what the family's kernels give."""
    from paper_1711_01348_amd import binding as B
    expr = make()
    w = wl.random_inputs(expr, 13)
    plan = B.Plan(expr)
    family = _run(plan, w, 0) if plan.workspace_bytes else None
    f_ref, g_ref = oracle.forward(expr, w.arg_list()), oracle.backward(expr, w.arg_list(), w.df)
    for how in (dict(null=True), dict(skew=4), dict(skew=1)):
        f, grads = _run(plan, w, max(plan.workspace_bytes, 64), **how)
        assert check.within(f, f_ref, expr.dtype) and all(check.within(g, r, expr.dtype) for g, r in zip(grads, g_ref)), how
        if family:
            assert np.array_equal(f, family[0]) and all(np.array_equal(g, r) for g, r in zip(grads, family[1])), how


def test_families_and_workspace_are_those_of_the_general_kernels():
    from paper_1711_01348_amd import binding as B
    e = wl.matmul_expr(100, 90, 70, "f64")
    assert B.Plan(e).forward_family == "generic" and B.Plan(e, generic_only=True).forward_family == "generic"
    e = wl.matmul_expr(40, 23, 5000, "f64")             # few tiles, long sum: partial sums
    assert B.Plan(e).workspace_bytes > B.Plan(e, generic_only=True).workspace_bytes


# tiles of every height, either orientation, sums that end in every part of the loop over stages of 32 (none, one, several stages with loads ahead,
# odd and even numbers, a partial last one); the last two: pieces of the sum
HEIGHTS = [(138, 379, 81, "f32"), (1621, 137, 39, "f32"), (611, 1631, 33, "f32"), (821, 577, 57, "f32"), (1173, 518, 65, "f32"), (927, 775, 25, "f32"),
           (1210, 673, 97, "f32"), (623, 1643, 27, "f32"), (743, 1607, 129, "f32"), (1303, 1293, 18, "f32"), (1127, 1477, 13, "f32"), (1999, 2003, 14, "f32"),
           (1871, 1601, 34, "f32"), (200, 941, 161, "f64"), (1449, 175, 38, "f64"), (538, 903, 193, "f64"), (825, 601, 61, "f64"), (488, 1155, 49, "f64"),
           (1595, 466, 31, "f64"), (1217, 1315, 225, "f64"), (1181, 906, 27, "f64"), (1141, 1110, 96, "f64"), (45, 51, 777, "f32"), (30, 1201, 640, "f64")]


@pytest.mark.gpu
@pytest.mark.parametrize("I,J,K,dtype", HEIGHTS)
def test_tiles_of_every_height(I, J, K, dtype):
    """Against numpy in 64 bits with the limits of check.py; 64-bit sums: within 16 units in the last place of the sum of the terms' magnitudes
    (chains of at most 16 + sqrt(K) additions, twice)."""
    from paper_1711_01348_amd import binding as B
    expr = wl.matmul_expr(I, J, K, dtype)
    w = wl.random_inputs(expr, 79)
    x, y = (a.astype(np.float64) for a in w.arg_list())
    d = w.df.astype(np.float64)
    f, (dx, dy) = _run(B.Plan(expr), w)
    for got, p, q in ((f, x, y), (dx, d, y.T), (dy, x.T, d)):
        ref = p @ q
        assert check.within(got, ref, dtype), check.errors(got, ref)
        if dtype == "f64":
            assert np.all(np.abs(got - ref) <= 16 * 2.0**-52 * (np.abs(p) @ np.abs(q)))


@pytest.mark.gpu
@pytest.mark.parametrize("I,J,K", [(1003, 701, 33), (1622, 137, 39), (137, 1622, 70), (2100, 1700, 19)])
def test_tiles_of_functions_and_with_an_outer_function(I, J, K):
    """Operands of either width, the outer function on tiles of either orientation."""
    from paper_1711_01348_amd import binding as B
    for expr in (wl.softplus_ratio_expr(I, J, K, "f32"), wl.dense_layer_expr(I, J, K, "f32")):
        w = wl.random_inputs(expr, 80)
        f, grads = _run(B.Plan(expr), w)
        assert check.within(f, oracle.forward(expr, w.arg_list()), "f32")
        for g, r in zip(grads, oracle.backward(expr, w.arg_list(), w.df)):
            assert check.within(g, r, "f32"), check.errors(g, r)


# every height of a tile: of plain products, with a program behind them, with column sums and scaled results beside them
HEIGHTS = [("matmul", 1433, 1190, 306, "f32"), ("matmul", 719, 1729, 381, "f32"), ("dense", 4710, 315, 76, "f32"), ("dense", 160, 4296, 83, "f32"),
           ("dense", 1500, 1024, 200, "f32"), ("dense", 2000, 300, 20, "f64"), ("matmul", 1077, 74, 14, "f32"),
           # ... where the model picks it for the sum, for sums in pieces, for one gradient and for both in a launch
           ("matmul", 716, 349, 16, "f32"), ("matmul", 905, 558, 18, "f32"), ("matmul", 1648, 930, 16, "f32"), ("matmul", 1924, 545, 17, "f32"),
           ("matmul", 879, 1729, 99, "f32"), ("matmul", 1129, 2765, 35, "f32"), ("matmul", 285, 345, 839, "f32"), ("matmul", 669, 593, 797, "f32"),
           ("matmul", 1098, 477, 16, "f64"), ("matmul", 631, 1203, 16, "f64"), ("matmul", 509, 2069, 16, "f64"), ("matmul", 250, 1055, 676, "f64"),
           ("matmul", 461, 524, 863, "f64"), ("matmul", 466, 429, 868, "f64"), ("matmul", 712, 529, 851, "f64"), ("dense", 420, 1832, 16, "f32"),
           ("dense", 2934, 468, 16, "f32"), ("dense", 541, 2853, 16, "f32"), ("dense", 354, 397, 647, "f32"), ("dense", 790, 736, 698, "f32"),
           ("dense", 457, 394, 875, "f64")]


@pytest.mark.gpu
@pytest.mark.parametrize("kind,M,N,K,dtype", HEIGHTS)
def test_heights_of_tiles(kind, M, N, K, dtype):
    import torch
    from paper_1711_01348_amd import binding as B, check
    e = dict(dense=wl.dense_layer_expr, matmul=wl.matmul_expr)[kind](M, N, K, dtype)
    w = wl.random_inputs(e, 17, -0.2, 0.2)
    plan = B.Plan(e)
    args = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in w.arg_list()]
    f = plan.forward(args)
    grads = plan.backward(args, f, torch.from_numpy(w.df).cuda())
    x, y = (a.astype(np.float64) for a in w.arg_list()[:2])
    df = w.df.astype(np.float64)
    f_ref = x @ y
    if kind == "dense":
        f_ref = np.tanh(f_ref + w.arg_list()[2].astype(np.float64))
        df = df * (1 - f_ref ** 2)
    refs = [f_ref, df @ y.T, x.T @ df] + ([df.sum(0)] if kind == "dense" else [])
    for g, r in zip([f] + list(grads), refs):
        assert check.within(g.cpu().numpy(), r, dtype), check.errors(g.cpu().numpy(), r)
