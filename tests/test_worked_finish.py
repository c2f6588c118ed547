"""Worked expression with a short sum: the launch that finishes the gradients - zeros of dc off its diagonal for any shape of c, columns with many tiles of rows."""
import pytest

from paper_1711_01348_amd import check
from paper_1711_01348_amd import workloads as wl


@pytest.mark.gpu
# tiles of rows up to 48, 192 and beyond, few columns; c as large as I x I, longer rows, more rows, rows a little longer than a workgroup's stores or shorter
@pytest.mark.parametrize("I,J,K,dtype,c_shape", [(3100, 9, 3, "f32", None), (3121, 70, 8, "f32", (3121, 3130)), (800, 33, 16, "f64", None), (3080, 3, 2, "f64", (3081, 3080)),
                                                 (40, 20, 2, "f32", (40, 1500)), (40, 20, 2, "f32", (1600, 41)), (17, 300, 5, "f64", (1021, 511)), (300, 5, 1, "f32", (301, 1023)),
                                                 (2900, 2900, 5, "f32", (2905, 2901)), (2897, 2900, 8, "f32", None),
                                                 # rows shorter than a workgroup's stores, than a store, of one element; many behind the diagonal's last one
                                                 (64, 40, 5, "f32", (9001, 64)), (600, 40, 3, "f32", (601, 603)), (3, 300, 3, "f32", (30001, 3)), (1, 40, 3, "f32", (9001, 1)),
                                                 (33, 20, 2, "f64", (4001, 33)), (2, 300, 3, "f64", (9001, 2)), (1, 300, 3, "f64", (3, 1))])
@pytest.mark.parametrize("before", [1, 4])   # a gradient of c that starts four or eight bytes off the alignment of the widest store, or on it
def test_finished_gradients(I, J, K, dtype, c_shape, before):
    import torch
    from paper_1711_01348_amd import binding as B
    expr = wl.worked_expr(I, J, K, dtype, c_shape=c_shape)
    dt = torch.float32 if dtype == "f32" else torch.float64
    g = torch.Generator(device="cuda")
    g.manual_seed(I + J + K)
    a, b, c, d = args = [torch.rand(tuple(q.shape), generator=g, device="cuda", dtype=dt) * s for q, s in zip(expr.args, (1.0, 1.0, 1.0 / K, 0.5))]
    df = torch.rand((I, J), generator=g, device="cuda", dtype=dt)
    plan = B.Plan(expr)
    f = plan.forward(args)
    # the gradient of c is watched on both sides
    room = torch.full((c.numel() + before + 1,), float("nan"), device="cuda", dtype=dt)
    out = [torch.full_like(a, float("nan")), torch.full_like(b, float("nan")), room[before:-1].view(c.shape), torch.full_like(d, float("nan"))]
    plan.backward(args, f, df, out=out)
    A, Bm, D3 = a.double(), b.double(), d.double() ** 3
    ci = c.diagonal()[:I].double()
    t = torch.exp(-(((A ** 2).sum(1)[:, None] + (Bm ** 2).sum(1)[None, :] + 2 * (A @ Bm.t().contiguous())) * ci[:, None] + D3.unfold(0, K, 1)[:I].sum(1)[:, None])) * df.double()
    r, P = t.sum(1), t @ Bm
    dd = torch.zeros_like(D3)
    for q in range(K):
        dd[q:q + I] += r
    want_dc = -((A ** 2).sum(1) * r + 2 * (A * P).sum(1) + t @ (Bm ** 2).sum(1))
    ct = ci[:, None] * t
    want = [-2 * ci[:, None] * (A * r[:, None] + P), -2 * (ct.t().contiguous() @ A + Bm * ct.sum(0)[:, None]), want_dc, -3 * d.double() ** 2 * dd]
    got = [out[0], out[1], out[2].diagonal()[:I], out[3]]
    for x, w in zip(got, want):
        # (every term of the gradients has one sign: the order of the sums costs a few roundings of the result)
        assert bool(((x.double() - w).abs() <= (2e-6 if dtype == "f32" else 1e-13) * w.abs() + 1e-30).all())
    rest = out[2].clone()
    rest.diagonal()[:I].zero_()
    assert not rest.any() and bool(room[:before].isnan().all()) and bool(room[-1].isnan())
