"""The entry point that allocates nothing (tad_eval_backward_static) against tad_eval_backward, through the C ABI."""
import ctypes

import numpy as np
import pytest

from paper_1711_01348_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _both(B, w):
    """Gradients of one workload from tad_eval_backward (caller's workspace) and from tad_eval_backward_static."""
    import torch
    plan = B.Plan(w.expr)
    n = len(w.expr.args)
    args = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in w.arg_list()]
    df = torch.from_numpy(w.df).cuda()
    f = plan.forward(args)
    ptrs = (ctypes.c_void_p * n)(*[t.data_ptr() for t in args])
    ws = plan.workspace()
    want = [torch.full_like(t, 3.0) for t in args]
    got = [torch.full_like(t, 5.0) for t in args]
    wptr = (ctypes.c_void_p * n)(*[t.data_ptr() for t in want])
    gptr = (ctypes.c_void_p * n)(*[t.data_ptr() for t in got])
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    assert B.lib.tad_eval_backward(plan._h, ptrs, f.data_ptr(), df.data_ptr(), wptr, ws.data_ptr(), ws.numel(), stream) == 0
    assert B.lib.tad_eval_backward_static(plan._h, ptrs, f.data_ptr(), df.data_ptr(), gptr, stream) == 0
    torch.cuda.synchronize()
    return plan, [t.cpu().numpy() for t in want], [t.cpu().numpy() for t in got]


def test_static_scratch_entry_point_matches_the_workspace_one():
    """Two calls in a row on the same GPU, the second with a smaller input (the array then still holds the partial
    sums of the first): both give exactly the gradients of tad_eval_backward, which the parity tests hold to the
    oracle.  A plan whose workspace exceeds the array is refused before anything is launched."""
    import torch
    from paper_1711_01348_amd import binding as B
    first = wl.random_inputs(wl.worked_expr(1024, 2048, 5, "f32"), 71, -0.8, 0.8)
    first.inputs["c"] = np.abs(first.inputs["c"]) * np.float32(0.2)
    second = wl.config3("small")
    sizes = []
    for w in (first, second, wl.config2(3, "small"), wl.config5("small")):
        plan, want, got = _both(B, w)
        assert 0 < plan.workspace_bytes <= B.STATIC_SCRATCH_BYTES
        sizes.append(plan.workspace_bytes)
        for a, x, y in zip(w.expr.args, want, got):
            assert np.array_equal(x, y), (w.name, "d" + a.name)
            assert not np.any(y == 5.0), (w.name, "d" + a.name, "not written")
    assert sizes[1] < sizes[0]
    # too large for the array: the 4096 x 4096 x 256 plan needs 64 MiB
    big = B.Plan(wl.config4().expr)
    assert big.workspace_bytes > B.STATIC_SCRATCH_BYTES
    four = (ctypes.c_void_p * 4)(*[1, 1, 1, 1])          # never dereferenced: the size check comes first
    assert B.lib.tad_eval_backward_static(big._h, four, 1, 1, four, None) == -7
    # the binding's switch reaches the same entry point
    w = second
    plan = B.Plan(w.expr)
    args = [torch.from_numpy(a).cuda() for a in w.arg_list()]
    f = plan.forward(args)
    df = torch.from_numpy(w.df).cuda()
    for x, y in zip(plan.backward(args, f, df), plan.backward(args, f, df, static=True)):
        assert torch.equal(x, y)


@pytest.mark.parametrize("make", [lambda: wl.dense_layer_expr(1500, 1024, 16, "f32"), lambda: wl.softplus_ratio_expr(1000, 500, 700, "f32")],
                         ids=["dense", "softplus"])
def test_a_plan_that_would_like_more_runs_on_the_kernels_that_do_with_less(make):
    """Accepted, the gradients of tad_eval_backward with a workspace as large as the array, and right."""
    import torch
    from paper_1711_01348_amd import binding as B, check
    expr = make()
    w = wl.random_inputs(expr, 31, -0.5, 0.5)
    plan = B.Plan(expr)
    assert plan.workspace_bytes > B.STATIC_SCRATCH_BYTES
    args = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in w.arg_list()]
    df = torch.from_numpy(w.df).cuda()
    f = plan.forward(args)
    ws = torch.empty(B.STATIC_SCRATCH_BYTES, dtype=torch.uint8, device="cuda")
    same, full = plan.backward(args, f, df, ws=ws), plan.backward(args, f, df)
    for a, s, x, y in zip(expr.args, plan.backward(args, f, df, static=True), same, full):
        assert torch.equal(s, x), a.name
        assert check.within(s.cpu().numpy(), y.cpu().numpy(), "f32"), a.name


# partial sums of products in pieces are a choice: they alone do not keep the dense products out of the array
@pytest.mark.parametrize("kind,M,N,K,dtype", [("dense", 320, 2701, 932, "f32"), ("dense", 481, 405, 5519, "f32"), ("dense", 535, 1043, 1732, "f32"),
                                              ("dense", 430, 1366, 684, "f64"), ("matmul", 3163, 2693, 98, "f32"), ("matmul", 6957, 1055, 104, "f32"),
                                              ("matmul", 2479, 2045, 237, "f64"), ("softplus", 282, 4919, 48, "f32")])
def test_dense_products_run_in_the_array(kind, M, N, K, dtype):
    """With fewer pieces where need be: the gradients of a workspace of any size from the array's to what the plan asks for."""
    import torch
    from paper_1711_01348_amd import binding as B, check
    expr = dict(dense=wl.dense_layer_expr, matmul=wl.matmul_expr, softplus=wl.softplus_ratio_expr)[kind](M, N, K, dtype)
    plan = B.Plan(expr)
    w = wl.random_inputs(expr, 32, -0.2, 0.2)
    args = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in w.arg_list()]
    df = torch.from_numpy(w.df).cuda()
    f = plan.forward(args)
    full = plan.backward(args, f, df)
    for static, n in ((True, None), (False, B.STATIC_SCRATCH_BYTES), (False, max(B.STATIC_SCRATCH_BYTES, plan.workspace_bytes - 1))):
        ws = None if static else torch.empty(n, dtype=torch.uint8, device="cuda")
        ms, launches = ctypes.c_double(0), ctypes.c_int(0)
        assert B.lib.tad_profile_begin(b"k_product", 1) == 0
        grads = plan.backward(args, f, df, static=True) if static else plan.backward(args, f, df, ws=ws)
        assert B.lib.tad_profile_end(ctypes.byref(ms), ctypes.byref(launches)) == 0
        assert launches.value >= 1
        for a, x, y in zip(expr.args, grads, full):
            assert check.within(x.cpu().numpy(), y.cpu().numpy(), dtype), a.name
    ws = torch.empty(B.STATIC_SCRATCH_BYTES, dtype=torch.uint8, device="cuda")
    assert check.within(plan.forward(args, ws=ws).cpu().numpy(), f.cpu().numpy(), dtype)
