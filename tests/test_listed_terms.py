"""Gradients whose terms are listed at plan time: the list in either of its forms."""
import numpy as np
import pytest

import oracle
from paper_1711_01348_amd import check
from paper_1711_01348_amd import workloads as wl
from paper_1711_01348_amd.workloads import ArgSpec, ExprSpec


def worked(I, J, K):
    return lambda dtype: wl.worked_expr(I, J, K, dtype)


def row_of(n):
    """tanh_dot of x_ik with a row of y: n + 8 elements."""
    return lambda dtype: ExprSpec("tanh_dot", (n // 8, 1), [(0, 7)], [ArgSpec("x", (n // 8, 8), [[1, 0, 0], [0, 0, 1]]),
                                                                       ArgSpec("y", (8, 1), [[0, 0, 1], [0, 1, 0]])], dtype)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f32", "f64"])
# elements of all gradients: few, 253, 285 (more than the short form has), 256, 264
@pytest.mark.parametrize("make", [worked(1, 1, 1), worked(8, 6, 5), worked(13, 4, 4), worked(14, 4, 4), row_of(248), row_of(256)],
                         ids=["1x1x1", "8x6x5", "13x4x4", "14x4x4", "256", "264"])
def test_either_form(make, dtype):
    import torch
    from paper_1711_01348_amd import binding as B
    expr = make(dtype)
    w = wl.random_inputs(expr, 31, -0.8, 0.8)
    plan = B.Plan(expr)
    args = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in w.arg_list()]
    f = plan.forward(args)
    grads = plan.backward(args, f, torch.from_numpy(w.df).cuda())
    assert check.within(f.cpu().numpy(), oracle.forward(expr, w.arg_list()), dtype)
    for a, g, r in zip(expr.args, grads, oracle.backward(expr, w.arg_list(), w.df)):
        assert check.within(g.cpu().numpy(), r, dtype), (a.name, check.errors(g.cpu().numpy(), r))
