"""Separable sums: the index maps of the passes over pairs of indices, as two indices with 32-bit steps or as they are."""
import pytest

import oracle
from paper_1711_01348_amd import check
from paper_1711_01348_amd import workloads as wl
from paper_1711_01348_amd.workloads import ArgSpec
from test_separable import A0, A1, A2, program, run


def unit(count, *d):
    return [[1 if c == q else 0 for c in range(count)] for q in d]


def extents_of_one(dtype):
    """x_{0i0k}, one contiguous index; y_{kj}, two."""
    I, J, K = 37, 18, 9
    return program((1, I, 1, J), [(0, K - 1)], [ArgSpec("x", (1, I, 1, K), unit(5, 0, 1, 2, 4)), ArgSpec("y", (K, J), unit(5, 4, 3))], dtype,
                   [A0, ("exp",), A1, ("cos",), ("mul",)], [("sum",)])


def one_of_two_operands_folds(dtype):
    """x_abk is one index by itself, u_{b+k} makes it three, v_ab keeps two."""
    a, b, J, K = 6, 5, 17, 11
    args = [ArgSpec("x", (a, b, K), unit(4, 0, 1, 3)), ArgSpec("y", (K, J), unit(4, 3, 2)), ArgSpec("u", (b + K - 1,), [[0, 1, 0, 1]])]
    return program((a, b, J), [(0, K - 1)], args, dtype, [A0, ("sin",), A2, ("mul",), A1, ("exp",), ("mul",)], [("sum",)])


def two_indices_behind_three(dtype):
    """x_abk w_ab: a and b are one index, k the other."""
    a, b, J, K = 4, 9, 16, 13
    args = [ArgSpec("x", (a, b, K), unit(4, 0, 1, 3)), ArgSpec("y", (J, K), unit(4, 2, 3)), ArgSpec("w", (a, b), unit(4, 0, 1))]
    return program((a, b, J), [(0, K - 1)], args, dtype, [A0, A2, ("mul",), ("exp",), A1, ("sin",), ("mul",)], [("sum",)])


def strided_windows(dtype):
    """x_{3i+2k} and y_{kj} of a larger tensor, transposed: steps that are not those of a tensor's own indices."""
    I, J, K = 40, 33, 20
    args = [ArgSpec("x", (3 * I + 2 * K,), [[3, 0, 2]]), ArgSpec("y", (J + 5, K + 3), [[0, 1, 0], [0, 0, 1]])]
    return program((I, J), [(0, K - 1)], args, dtype, [A0, ("exp",), A1, ("sin",), ("mul",)], [("sum",)])


def a_long_function(dtype):
    """A program of more than one line of operations, with constants of at most 1: no operation enlarges the rounding of the one before.  (With
    factors up to 3.5 the 32-bit terms of the general kernels may be off by the product of all factors, 170 units: they were, by 1e-4 where
    the value is near 0.)"""
    I, J, K = 33, 20, 16
    inner = [A0]
    for n in range(8):
        inner += [("const", 0.25 + n % 4 / 4), ("mul",), ("sin",)]
    args = [ArgSpec("x", (I, K), unit(3, 0, 2)), ArgSpec("y", (K, J), unit(3, 2, 1))]
    return program((I, J), [(0, K - 1)], args, dtype, inner + [A1, ("exp",), ("mul",)], [("sum",), ("tanh",)])


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("make", [extents_of_one, one_of_two_operands_folds, two_indices_behind_three, strided_windows, a_long_function])
def test_index_maps(make, dtype):
    from paper_1711_01348_amd import binding as B
    expr = make(dtype)
    w = wl.random_inputs(expr, 23, -0.8, 0.8)
    plan, general = B.Plan(expr), B.Plan(expr, generic_only=True)
    for ws_bytes in (None, general.workspace_bytes):
        f, grads = run(plan, w, ws_bytes)
        assert check.within(f, oracle.forward(expr, w.arg_list()), dtype)
        for a, g, r in zip(expr.args, grads, oracle.backward(expr, w.arg_list(), w.df)):
            assert check.within(g, r, dtype), (a.name, check.errors(g, r))
