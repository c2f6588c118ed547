"""Strided family: gradients by pairs (i, j), for every number of pairs per thread, by columns, and at the edges of the rule between them."""
import numpy as np
import pytest

import oracle
from paper_1711_01348_amd import check
from paper_1711_01348_amd import workloads as wl


def _run(expr, inputs, wanted=None):
    import torch
    from paper_1711_01348_amd import binding as B
    plan = B.Plan(expr)
    assert plan.forward_family == "strided"
    args = [torch.from_numpy(a).cuda() for a in inputs.arg_list()]
    f = plan.forward(args)
    grads = plan.backward(args, f, torch.from_numpy(inputs.df).cuda(), wanted=wanted)
    torch.cuda.synchronize()
    return f.cpu().numpy(), [None if g is None else g.cpu().numpy() for g in grads]


# one, two, four and eight pairs per thread with ragged last rows; rows of 255, 256, 257 and more than 1024 pairs;
# more than a workgroup's LDS (by columns); a stride above the number of taps; strides 8 and 9
CASES = [(2, 6, 5, 3, 3, 2), (3, 4, 254, 3, 2, 1), (3, 4, 255, 3, 2, 1), (3, 4, 256, 3, 2, 1), (64, 40, 33, 2, 2, 1), (32, 70, 61, 3, 3, 2),
         (32, 65, 130, 3, 3, 2), (96, 33, 65, 2, 2, 1), (1, 5, 1023, 2, 2, 1), (1, 3, 1500, 3, 3, 1), (1, 9, 700, 7, 7, 3), (2, 5, 9, 2, 2, 5), (2, 5, 9, 3, 3, 8), (2, 5, 9, 3, 3, 9),
         (4, 1, 1, 1, 1, 1), (1, 3, 20, 49, 1, 1), (1, 20, 3, 1, 49, 2)]


@pytest.mark.gpu
@pytest.mark.parametrize("N,I,J,U,V,stride", CASES)
def test_gradients_of_every_split(N, I, J, U, V, stride):
    expr = wl.strided_tanh_expr(N, I, J, U, V, stride, "f32")
    inputs = wl.random_inputs(expr, 5, -0.3, 0.3)
    f, grads = _run(expr, inputs)
    assert check.within(f, oracle.forward(expr, inputs.arg_list()), "f32")
    reference = oracle.backward(expr, inputs.arg_list(), inputs.df)
    for g, r in zip(grads, reference):
        assert check.within(g, r, "f32"), check.errors(g, r)
    for only in (0, 1):
        _, alone = _run(expr, inputs, wanted=[only == 0, only == 1])
        assert alone[1 - only] is None
        assert np.array_equal(alone[only], grads[only])


@pytest.mark.gpu
@pytest.mark.parametrize("value", [np.inf, np.nan])
def test_terms_that_do_not_exist_are_left_out(value):
    """A tap that is no number reaches the elements of dx that have a term with it, and no others."""
    expr = wl.strided_tanh_expr(2, 7, 9, 3, 3, 1, "f32")
    inputs = wl.random_inputs(expr, 6, 0.1, 0.4)
    f = oracle.forward(expr, inputs.arg_list())
    args = [a.copy() for a in inputs.arg_list()]
    args[1][0, 0] = value        # read by p < 7, q < 9 only
    import torch
    from paper_1711_01348_amd import binding as B
    plan = B.Plan(expr)
    on = [torch.from_numpy(a).cuda() for a in args]
    dx = plan.backward(on, torch.from_numpy(f.astype(np.float32)).cuda(), torch.from_numpy(inputs.df).cuda())[0].cpu().numpy()
    finite = np.isfinite(dx)
    assert finite[:, 7:, :].all() and finite[:, :, 9:].all() and not finite[:, :7, :9].any()


@pytest.mark.gpu
def test_infinite_inputs_stay_with_their_own_terms():
    """Elements of x that no function index reads beyond the last window do not reach dw."""
    expr = wl.strided_tanh_expr(2, 6, 7, 2, 2, 3, "f32")
    inputs = wl.random_inputs(expr, 7, -0.3, 0.3)
    args = [a.copy() for a in inputs.arg_list()]
    args[0][:, 2::3, :] = np.inf      # rows between the windows
    import torch
    from paper_1711_01348_amd import binding as B
    plan = B.Plan(expr)
    f = oracle.forward(expr, inputs.arg_list()).astype(np.float32)
    dw = plan.backward([torch.from_numpy(a).cuda() for a in args], torch.from_numpy(f).cuda(), torch.from_numpy(inputs.df).cuda())[1]
    r = oracle.backward(expr, inputs.arg_list(), inputs.df)[1]
    assert check.within(dw.cpu().numpy(), r, "f32")


# by columns: two taps at most in a direction, or more; strides on either side of the rule, from its smallest tensor on; a filter taller than a
# workgroup's rows; rows of f longer than a workgroup takes for dw; few elements to a workgroup; more images than a grid has along its second axis
COLUMNS = [(2, 5, 9, 7, 7, 4), (2, 5, 9, 7, 7, 3), (1, 6, 11, 9, 5, 4), (3, 4, 5, 3, 3, 16), (2, 3, 70, 1, 1, 5), (2, 4, 7, 16, 3, 5), (1, 2, 300, 3, 3, 4),
           (1, 300, 2, 1, 7, 4), (16, 127, 129, 3, 3, 2), (17, 127, 129, 3, 3, 2), (9, 119, 121, 5, 5, 2), (2, 200, 70, 49, 1, 1), (1, 3, 1030, 2, 2, 4),
           (40, 9, 28, 3, 3, 1), (40, 9, 28, 7, 7, 1), (65536, 2, 1, 1, 2, 1), (65537, 1, 2, 2, 2, 3)]


@pytest.mark.gpu
@pytest.mark.parametrize("N,I,J,U,V,stride", COLUMNS)
def test_gradients_by_columns(N, I, J, U, V, stride):
    """Also with rows and columns of x behind the last term, where the gradient is zero."""
    for more in (0, 3):
        expr = wl.strided_tanh_expr(N, I, J, U, V, stride, "f32")
        x = expr.args[0]
        x.shape = (x.shape[0], x.shape[1] + more, x.shape[2] + more)
        if x.shape[0] * x.shape[1] * x.shape[2] > 1 << 22:
            continue
        inputs = wl.random_inputs(expr, 8, -0.3, 0.3)
        f, grads = _run(expr, inputs)
        assert check.within(f, oracle.forward(expr, inputs.arg_list()), "f32")
        for g, r in zip(grads, oracle.backward(expr, inputs.arg_list(), inputs.df)):
            assert check.within(g, r, "f32"), check.errors(g, r)
            assert np.all(g[r == 0] == 0)
        for only in (0, 1):
            _, alone = _run(expr, inputs, wanted=[only == 0, only == 1])
            assert np.array_equal(alone[only], grads[only])


@pytest.mark.gpu
@pytest.mark.parametrize("U,stride", [(3, 4), (9, 4)])
def test_terms_that_do_not_exist_are_left_out_by_columns(U, stride):
    """A tap that is no number reaches the elements of dx that have a term with it, and no others."""
    import torch
    from paper_1711_01348_amd import binding as B
    I, J = 5, 6
    expr = wl.strided_tanh_expr(2, I, J, U, 5, stride, "f32")
    inputs = wl.random_inputs(expr, 9, 0.1, 0.4)
    f = oracle.forward(expr, inputs.arg_list()).astype(np.float32)
    args = [a.copy() for a in inputs.arg_list()]
    args[1][U - 1, 4] = np.inf
    plan = B.Plan(expr)
    dx = plan.backward([torch.from_numpy(a).cuda() for a in args], torch.from_numpy(f).cuda(), torch.from_numpy(inputs.df).cuda())[0].cpu().numpy()
    reached = np.zeros(dx.shape, dtype=bool)
    reached[:, U - 1:U - 1 + stride * (I - 1) + 1:stride, 4:4 + stride * (J - 1) + 1:stride] = True
    assert np.array_equal(~np.isfinite(dx), reached)
