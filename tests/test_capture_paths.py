"""The paths chosen beside a plan's family, recorded into a graph: every replay gives what the eager calls give."""
import pytest

from paper_1711_01348_amd import workloads as wl

pytestmark = pytest.mark.gpu


def matmul(I, J, K, dtype):
    return wl.matmul_expr(I, J, K, dtype)


CASES = [("separable", lambda: wl.softplus_ratio_expr(70, 65, 33, "f32")), ("separable_from_f", lambda: wl.dense_layer_expr(64, 16, 1100, "f64")),
         ("product_pieces", lambda: matmul(40, 23, 1100, "f32")), ("worked_wide", lambda: wl.worked_expr(130, 65, 3, "f32")),
         ("index_sum_wide", lambda: wl.index_sum_exp_expr(517, 999, "f32")), ("conditions", lambda: wl.causal_convolution_expr(70, 9, "f32")),
         ("bf16_parts", lambda: matmul(4100, 2052, 1028, "f32")), ("worked_long", lambda: wl.worked_expr(2049, 3900, 128, "f32"))]


@pytest.mark.parametrize("name,make", CASES, ids=[c[0] for c in CASES])
def test_replays_match_eager_calls(name, make):
    import torch
    from paper_1711_01348_amd import binding as B
    expr = make()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    dt = torch.float64 if expr.dtype == "f64" else torch.float32
    draw = lambda shape: torch.rand(tuple(shape), generator=gen, dtype=dt, device="cuda") - 0.5
    plan, args, df = B.Plan(expr), [draw(a.shape) for a in expr.args], draw(expr.f_shape)
    f, out, ws = torch.empty_like(df), [torch.empty_like(a) for a in args], plan.workspace()

    def step():
        plan.forward(args, out=f, ws=ws)
        plan.backward(args, f, df, out=out, ws=ws)

    step()
    torch.cuda.synchronize()
    want = [t.clone() for t in [f] + out]
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        step()
    side.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        step()
    for _ in range(3):
        for t in [f] + out:
            t.fill_(float("nan"))
        ws.fill_(255)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for t, w in zip([f] + out, want):
            assert torch.equal(t, w)
        step()                                   # the program's own work between the replays
        torch.cuda.synchronize()
