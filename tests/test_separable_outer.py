"""Separable sums: the pass that applies a function of the result alone takes several elements per thread."""
import pytest

import oracle
from paper_1711_01348_amd import check
from paper_1711_01348_amd import workloads as wl
from test_separable import run


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f32", "f64"])
# results: fewer than a workgroup's (1024, 512 in 64 bits), one less, as many, one more, several workgroups and a remainder
@pytest.mark.parametrize("M,N", [(16, 16), (31, 33), (32, 32), (25, 41), (16, 33), (65, 67)])
def test_gradients_of_a_dense_layer(M, N, dtype):
    from paper_1711_01348_amd import binding as B
    w = wl.random_inputs(wl.dense_layer_expr(M, N, 9, dtype), 5, -0.8, 0.8)
    plan = B.Plan(w.expr)
    f, grads = run(plan, w)
    assert check.within(f, oracle.forward(w.expr, w.arg_list()), dtype)
    for a, g, r in zip(w.expr.args, grads, oracle.backward(w.expr, w.arg_list(), w.df)):
        assert check.within(g, r, dtype), (a.name, check.errors(g, r))


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f32", "f64"])
# tiles of 16, 32 and more rows, each with remainders in rows and columns: what the program reads is fetched before or behind the sum
@pytest.mark.parametrize("M,N,K", [(1, 1, 3), (17, 129, 40), (130, 515, 33), (515, 387, 9), (1030, 1030, 5)])
def test_low_and_tall_tiles_apply_the_same_program(M, N, K, dtype):
    from paper_1711_01348_amd import binding as B
    w = wl.random_inputs(wl.dense_layer_expr(M, N, K, dtype), 6, -0.8, 0.8)
    plan = B.Plan(w.expr)
    f, grads = run(plan, w)
    assert check.within(f, oracle.forward(w.expr, w.arg_list()), dtype)
    for a, g, r in zip(w.expr.args, grads, oracle.backward(w.expr, w.arg_list(), w.df)):
        assert check.within(g, r, dtype), (a.name, check.errors(g, r))
