"""Separable sums: gradients as products whose results are multiplied by partial derivatives that were evaluated with the factors."""
import numpy as np
import pytest

import oracle
from paper_1711_01348_amd import check
from paper_1711_01348_amd import workloads as wl
from paper_1711_01348_amd.workloads import ArgSpec, ExprSpec

A = [("arg", p) for p in range(6)]
X, Y, Z = [[1, 0, 0], [0, 0, 1]], [[0, 0, 1], [0, 1, 0]], [[1, 0, 1]]


def _expr(I, J, K, dtype, inner, outer, extra):
    args = [ArgSpec("x", (I, K), X), ArgSpec("y", (K, J), Y)]
    args += [ArgSpec(f"u{n}", (I, K) if kind == "pair" else (I + K - 1,), X if kind == "pair" else Z) for n, kind in enumerate(extra)]
    return ExprSpec("program", (I, J), [(0, K - 1)], args, dtype, inner, outer)


# The outer function reads the sum rounded to 32 bits, so it is one that does not make more of that: the logarithm of 1 + s, s > 0, changes
# by at most 2^-24 s / (1 + s) for it (a sine of s = 40 by 2.4e-6).
def value_is_derivative(I, J, K):     # exp(x) sqrt(y^2 + 1): one result for x's side
    return _expr(I, J, K, "f32", [A[0], ("exp",), A[1], ("powi", 2), ("const", 1.0), ("add",), ("sqrt",), ("mul",)], [("const", 1.0), ("sum",), ("add",), ("log",)], [])


def two_of_a_side(I, J, K):           # x: an element per pair, u: a window
    return _expr(I, J, K, "f32", [A[0], ("sin",), A[2], ("cos",), ("mul",), A[1], ("exp",), ("mul",)], [("sum",)], ["window"])


def two_elements_per_pair(I, J, K):   # both would be stored in the same place: the derivative of the factor is
    return _expr(I, J, K, "f32", [A[0], A[2], ("mul",), ("exp",), A[1], ("sin",), ("mul",)], [("sum",)], ["pair"])


def three_of_a_side(I, J, K):
    return _expr(I, J, K, "f32", [A[0], ("exp",), A[2], ("mul",), A[3], ("cos",), ("mul",), A[1], ("mul",)], [("sum",)], ["window", "window"])


def same_derivative(I, J, K):         # d / dx and d / du are the same operation
    return _expr(I, J, K, "f32", [A[0], A[2], ("add",), ("sin",), A[1], ("cos",), ("mul",)], [("sum",)], ["window"])


def constant_derivative(I, J, K):     # no operation yields d / dx
    return _expr(I, J, K, "f32", [A[0], ("const", 1.5), ("add",), A[1], ("exp",), ("mul",)], [("sum",)], [])


def no_registers(I, J, K):            # x's factor has more live values than registers, y's has a program of two results
    inner = []
    for p in (0, 2):
        for fn in [("exp",), ("sin",), ("cos",), ("tanh",), ("neg",), ("powi", 2), ("powi", 3), ("powi", 4), ("powi", 5)]:
            inner += [A[p], fn]
    return _expr(I, J, K, "f32", inner + [("add",)] * 17 + [A[1], ("sin",), ("mul",)], [("sum",)], ["window"])


def wide(I, J, K):
    return _expr(I, J, K, "f64", [A[0], ("exp",), A[1], ("sin",), ("mul",)], [("sum",), ("powi", 2)], [])


MAKES = [value_is_derivative, two_of_a_side, two_elements_per_pair, three_of_a_side, same_derivative, constant_derivative, no_registers, wide]


@pytest.mark.gpu
# tiles of 16 x 64 with ragged edges; both gradients in a launch or one each; sums long enough for pieces
@pytest.mark.parametrize("I,J,K", [(16, 17, 9), (70, 65, 33), (16, 2000, 40), (130, 140, 70)])
@pytest.mark.parametrize("make", MAKES, ids=[m.__name__ for m in MAKES])
def test_scaled_gradients(make, I, J, K):
    import torch
    from paper_1711_01348_amd import binding as B
    expr = make(I, J, K)
    w = wl.random_inputs(expr, 17, -0.8, 0.8)
    plan = B.Plan(expr)
    args = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in w.arg_list()]
    df = torch.from_numpy(w.df).cuda()
    ws = torch.full((plan.workspace_bytes + 16,), 255, dtype=torch.uint8, device="cuda")   # NaNs: nothing is read before it is written
    f = plan.forward(args, ws=ws)
    grads = plan.backward(args, f, df, ws=ws)
    torch.cuda.synchronize()
    assert check.within(f.cpu().numpy(), oracle.forward(expr, w.arg_list()), expr.dtype)
    reference = oracle.backward(expr, w.arg_list(), w.df)
    for a, g, r in zip(expr.args, grads, reference):
        assert check.within(g.cpu().numpy(), r, expr.dtype), (a.name, check.errors(g.cpu().numpy(), r))
    for only in range(len(args)):     # some gradients of a side and not the others
        ws.fill_(255)
        alone = plan.backward(args, f, df, wanted=[p == only for p in range(len(args))], ws=ws)[only].cpu().numpy()
        assert check.within(alone, reference[only], expr.dtype), (only, check.errors(alone, reference[only]))


@pytest.mark.gpu
# fewer rows than threads to a column, one batch and more than one, either side of the line; columns that do not fill a workgroup's
@pytest.mark.parametrize("I,J,K", [(17, 16, 9), (31, 33, 20), (256, 17, 16), (257, 250, 40), (4096, 18, 16), (4097, 18, 16), (6144, 18, 16), (6145, 18, 16)])
@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_bias_gradients_beside_the_products(I, J, K, dtype):
    import torch
    from paper_1711_01348_amd import binding as B
    expr = wl.dense_layer_expr(I, J, K, dtype)
    w = wl.random_inputs(expr, 23, -0.5, 0.5)
    plan = B.Plan(expr)
    args = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in w.arg_list()]
    df, ws = torch.from_numpy(w.df).cuda(), plan.workspace()
    f = plan.forward(args, ws=ws)
    reference = oracle.backward(expr, w.arg_list(), w.df)
    n = len(args)
    # all of them; the bias with one factor; the bias alone (no product to go with)
    for wanted in ([True] * n, [True] + [False] * (n - 2) + [True], [False] * (n - 1) + [True]):
        grads = plan.backward(args, f, df, wanted=wanted, ws=ws)
        for a, g, r, is_wanted in zip(expr.args, grads, reference, wanted):
            assert (g is not None) == is_wanted
            if is_wanted:
                assert check.within(g.cpu().numpy(), r, dtype), (a.name, check.errors(g.cpu().numpy(), r))
