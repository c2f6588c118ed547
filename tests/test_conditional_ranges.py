"""Sums whose extra conditions bound the last summation index: the forward kernels turn them into a range of the run."""
import numpy as np
import pytest

import oracle
from paper_1711_01348_amd import check
from paper_1711_01348_amd import workloads as wl
from paper_1711_01348_amd.workloads import ArgSpec, ExprSpec


def two_index(dtype):
    """Coefficients above one in either direction, a condition without the last index, lower limits that are not zero, function
    indices without any term."""
    return ExprSpec("mul", (23,), [(1, 4), (2, 17)], [ArgSpec("x", (23, 18), [[1, 0, 0], [0, 0, 1]]), ArgSpec("y", (5, 18), [[0, 1, 0], [0, 0, 1]])],
                    dtype, constraints=[([1, 0, -3], 7), ([-1, 2, 2], -3), ([2, -5, 0], 1)])


def one_index(dtype):
    return ExprSpec("exp", (40,), [(3, 90)], [ArgSpec("x", (40, 91), [[1, 0], [0, 1]])], dtype, constraints=[([-2, 5], -31), ([1, -2], 95)])


def outside(dtype):
    """No term at all for half of the function indices."""
    return ExprSpec("tanh_dot", (30,), [(0, 8)], [ArgSpec("x", (30, 9), [[1, 0], [0, 1]]), ArgSpec("w", (9,), [[0, 1]])], dtype,
                    constraints=[([1, 1], -15)])


CASES = [(f.__name__, f) for f in (two_index, one_index, outside)]
CASES += [("causal", lambda dt: wl.causal_convolution_expr(70, 9, dt)), ("causal_wide", lambda dt: wl.causal_convolution_expr(9, 9, dt)),
          ("cumulative_long", lambda dt: wl.cumulative_sum_expr(2100, dt, "exp"))]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("name,make", CASES, ids=[c[0] for c in CASES])
def test_conditions_as_ranges(name, make, dtype):
    """Built-in body and the same written as a program, against the oracle."""
    import torch
    from paper_1711_01348_amd import binding as B
    expr = make(dtype)
    scale = 0.02 if "cumulative" in name else 0.2 if expr.body == "exp" else 1.0
    w = wl.random_inputs(expr, 31, -scale, scale)
    f_ref, g_ref = oracle.forward(expr, w.arg_list()), oracle.backward(expr, w.arg_list(), w.df)
    args, df = [torch.from_numpy(a).cuda() for a in w.arg_list()], torch.from_numpy(w.df).cuda()
    for plan in (B.Plan(expr), B.Plan(wl.as_program(expr), keep_program=True)):
        f = plan.forward(args)
        grads = plan.backward(args, f, df)
        torch.cuda.synchronize()
        assert check.within(f.cpu().numpy(), f_ref, dtype), check.errors(f.cpu().numpy(), f_ref)
        for g, r in zip(grads, g_ref):
            assert check.within(g.cpu().numpy(), r, dtype), check.errors(g.cpu().numpy(), r)
            assert np.all(g.cpu().numpy()[r == 0] == 0)
