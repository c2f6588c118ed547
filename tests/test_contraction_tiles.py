"""Products of 32-bit matrices on the 32-bit matrix instructions: tiles of 64 x 64 at their edges, every memory order."""
import numpy as np
import pytest

from paper_1711_01348_amd import workloads as wl


@pytest.mark.gpu
@pytest.mark.parametrize("xt,yt", [(False, False), (True, False), (False, True), (True, True)])
# one tile short of and beyond 64, a contraction index of one load and behind a whole tile, pieces of the sum
@pytest.mark.parametrize("I,J,K", [(1276, 1220, 4), (1284, 1216, 36), (700, 644, 604), (64, 4100, 1028), (60, 2052, 2260)])
def test_products(I, J, K, xt, yt):
    import torch
    from paper_1711_01348_amd import binding as B
    expr = wl.matmul_expr(I, J, K, "f32", xt, yt)
    plan = B.Plan(expr)
    assert plan.forward_family == "contraction"
    w = wl.random_inputs(expr, 31)
    x, y = (torch.from_numpy(a) for a in w.arg_list())
    df = torch.from_numpy(w.df)
    f = plan.forward([x.cuda(), y.cuda()])
    grads = plan.backward([x.cuda(), y.cuda()], f, df.cuda())
    X, Y, D = (x.t() if xt else x).double(), (y.t() if yt else y).double(), df.double()
    back = lambda t, turned: t.t() if turned else t
    for got, (p, q), turned in ((f, (X, Y), False), (grads[0], (D, Y.t()), xt), (grads[1], (X.t(), D), yt)):
        exact, size = back(p @ q, turned), back(p.abs() @ q.abs(), turned)
        # n products and n - 1 additions, one rounding each (in any order), and the result's
        bound = (p.shape[1] + 2) * 2.0 ** -24 * size
        assert bool(((got.cpu().double() - exact).abs() <= bound).all())


@pytest.mark.gpu
# either side of the rule for tiles of 128 x 128: 480 of them with ragged edges, 464, a sum of one stage less
@pytest.mark.parametrize("I,J,K", [(2045, 3836, 256), (1920, 3700, 256), (2045, 3836, 224), (130, 32636, 288)])
def test_forward_tiles_of_the_worked_expression(I, J, K):
    import torch
    from paper_1711_01348_amd import binding as B, check
    expr = wl.worked_expr(I, J, K, "f32")
    plan = B.Plan(expr)
    assert plan.forward_family == "worked_mfma"
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    a, b, c, d = [(torch.rand(tuple(q.shape), generator=g, device="cuda") - 0.5) * s for q, s in zip(expr.args, (2.0, 2.0, 1.0 / K, 0.4))]
    f = torch.full((I, J), float("nan"), device="cuda")
    plan.forward([a, b, c, d], out=f)
    A, Bm, D3 = a.double(), b.double(), d.double() ** 3
    s = (A ** 2).sum(1)[:, None] + (Bm ** 2).sum(1)[None, :] + 2 * (A @ Bm.t())
    window = torch.stack([D3[k:k + I] for k in range(K)]).sum(0)
    want = torch.exp(-(s * c.diagonal()[:I].double()[:, None] + window[:, None]))
    assert check.within(f.cpu().numpy(), want.cpu().numpy(), "f32"), check.errors(f.cpu().numpy(), want.cpu().numpy())
