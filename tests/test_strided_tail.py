"""Strided family: slices of f that go on behind the end of a tensor whose size is not a multiple of the vector width."""
import numpy as np
import pytest

import oracle
from paper_1711_01348_amd import check
from paper_1711_01348_amd import workloads as wl


@pytest.mark.gpu
@pytest.mark.parametrize("N,I,J,U,V,stride", [(9, 27, 9, 3, 3, 1), (3, 21, 37, 3, 3, 1), (1, 9, 11, 3, 3, 1), (5, 17, 7, 2, 2, 1),
                                              (7, 13, 5, 5, 5, 2), (2, 23, 19, 7, 7, 1), (1, 3, 1, 3, 3, 1)])
def test_gradient_at_the_tail_of_a_ragged_tensor(N, I, J, U, V, stride):
    import torch
    from paper_1711_01348_amd import binding as B
    expr = wl.strided_tanh_expr(N, I, J, U, V, stride, "f32")
    w = wl.random_inputs(expr, 3, -0.4, 0.4)
    plan = B.Plan(expr)
    assert plan.forward_family == "strided"
    args = [torch.from_numpy(a).cuda() for a in w.arg_list()]
    f = plan.forward(args)
    grads = plan.backward(args, f, torch.from_numpy(w.df).cuda())
    torch.cuda.synchronize()
    assert check.within(f.cpu().numpy(), oracle.forward(expr, w.arg_list()), "f32")
    for g, r in zip(grads, oracle.backward(expr, w.arg_list(), w.df)):
        assert check.within(g.cpu().numpy(), r, "f32"), check.errors(g.cpu().numpy(), r)
