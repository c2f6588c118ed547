"""Worked expression with a long sum: contractions on the bf16 matrix cores and on the 32-bit ones, in pieces of any number, against 64 bits."""
import ctypes

import pytest

from paper_1711_01348_amd import check
from paper_1711_01348_amd import workloads as wl

pytestmark = pytest.mark.gpu


def tensors(I, J, K, seed=3, c_extra=0):
    import torch
    expr = wl.worked_expr(I, J, K, "f32", c_shape=(I + c_extra, I + c_extra + 1) if c_extra else None)
    g = torch.Generator(device="cuda")
    g.manual_seed(seed + I + J + K)
    args = [(torch.rand(tuple(q.shape), generator=g, device="cuda") - 0.5) * s for q, s in zip(expr.args, (2.0, 2.0, 1.0 / K, 0.4))]
    return expr, args, torch.rand((I, J), generator=g, device="cuda") * 2 - 1


def evaluate(plan, args, df, ws_bytes, wanted=(0, 1, 2, 3), f=None):
    """f and the wanted gradients with ws_bytes of workspace, everything behind it watched; gradients of a given f if there is one."""
    import torch
    from paper_1711_01348_amd import binding as B
    out, grads = torch.full_like(df, float("nan")), [torch.full_like(a, float("nan")) for a in args]
    ws = torch.full((ws_bytes + 4096,), 255, dtype=torch.uint8, device="cuda")
    ptrs = (ctypes.c_void_p * 4)(*[t.data_ptr() for t in args])
    outs = (ctypes.c_void_p * 4)(*[t.data_ptr() if q in wanted else None for q, t in enumerate(grads)])
    assert B.lib.tad_eval_forward(plan._h, ptrs, out.data_ptr(), ws.data_ptr(), ws_bytes, None) == 0
    f = out if f is None else f
    assert B.lib.tad_eval_backward(plan._h, ptrs, f.data_ptr(), df.data_ptr(), outs, ws.data_ptr(), ws_bytes, None) == 0
    torch.cuda.synchronize()
    assert bool((ws[ws_bytes:] == 255).all()), "written beyond the workspace"
    return [out] + [grads[q] for q in wanted]


def exact(args, df, K, given=None):
    """f and the gradients in 64 bits, those of a given f if there is one."""
    import torch
    a, b, c, d = [t.double() for t in args]
    df, I = df.double(), df.shape[0]
    ci, na, nb = c.diagonal()[:I], (a * a).sum(1), (b * b).sum(1)
    f = torch.exp(-(ci[:, None] * (na[:, None] + nb[None, :] + 2 * (a @ b.t().contiguous())) + (d ** 3).unfold(0, K, 1)[:I].sum(1)[:, None]))
    g = df * (f if given is None else given.double())
    r, P = g.sum(1), g @ b
    dc, dd = torch.zeros_like(c), torch.zeros_like(d)
    dc.diagonal()[:I].copy_(-(na * r + 2 * (a * P).sum(1) + g @ nb))
    for q in range(K):
        dd[q:q + I] += r
    db = -2 * ((ci[:, None] * g).t().contiguous() @ a + b * (ci[:, None] * g).sum(0)[:, None])
    return [f, -2 * ci[:, None] * (a * r[:, None] + P), db, dc, -3 * d * d * dd]


def errors(tensors, want):
    return [((t.double() - w).norm() / w.norm()).item() for t, w in zip(tensors, want)]


# 64, 128 and 256 columns of a tile, a part of them and more than one; rows and terms one beyond a tile, a stage, four of them short; the forward pass on the bf16
# matrix cores as well, with sums of 128 to 512 terms
@pytest.mark.parametrize("I,J,K,c_extra,forward", [(1025, 1024, 32, 3, False), (1150, 1028, 64, 0, False), (1537, 1284, 96, 0, False), (1409, 1412, 128, 1, False),
                                                   (1409, 1540, 160, 0, False), (1921, 1148, 256, 0, False), (4097, 516, 288, 0, False), (509, 4100, 512, 2, False),
                                                   (2049, 4000, 160, 0, True), (2049, 4000, 128, 0, True), (2433, 3076, 256, 1, True), (2817, 2700, 512, 0, True)])
def test_error_is_no_larger_than_that_of_the_32_bit_kernels(I, J, K, c_extra, forward):
    """f, da and db are products.  dc and dd are mostly sums beside them, made alike in pieces of other lengths: dc within a tenth, dd, where a few roundings of
    long windows decide, within a factor of two (0.8 to 1.5 over sizes and inputs)."""
    import torch
    from paper_1711_01348_amd import binding as B
    expr, args, df = tensors(I, J, K, c_extra=c_extra)
    plan, want = B.Plan(expr), exact(args, df, K)
    split, plain = (evaluate(plan, args, df, n) for n in (plan.workspace_bytes, plan.workspace_bytes - 16))
    assert not torch.equal(split[1], plain[1]) and torch.equal(split[0], plain[0]) == (not forward)      # not the same kernels
    for e, p, limit, s, w in zip(errors(split, want), errors(plain, want), (1.02, 1.02, 1.02, 1.1, 2), split, want):
        assert e <= limit * p, (e, p)
        assert check.within(s.cpu().numpy(), w.cpu().numpy(), "f32"), check.errors(s.cpu().numpy(), w.cpu().numpy())
    rest = split[3].clone()
    rest.diagonal()[:I].zero_()
    assert not rest.any()


# small numbers: what they do to a, b, df and a given f
SMALL = {"df": lambda a, b, df, f: (a, b, df * 2.0 ** -115, None), "decayed_f": lambda a, b, df, f: (a, b, df, f * 2.0 ** -118),
         "a_and_b": lambda a, b, df, f: (a * 2.0 ** -118, b * 2.0 ** -118, df * 2.0 ** 60, None),
         "denormals": lambda a, b, df, f: (a * 2.0 ** 24, b * 2.0 ** 24, df * 2.0 ** -130, f)}


@pytest.mark.parametrize("I,J,K", [(1150, 1028, 64), (1409, 1540, 128), (1921, 1148, 256)])
@pytest.mark.parametrize("small", SMALL)
def test_small_numbers_are_not_less_exact_than_on_the_32_bit_kernels(I, J, K, small):
    """da, db, dc, which take products, against 64 bits (dc of the third kind, 2^-176, is 0 in 32 bits)."""
    import torch
    from paper_1711_01348_amd import binding as B
    expr, (a, b, c, d), df = tensors(I, J, K)
    g = torch.Generator(device="cuda")
    g.manual_seed(4)
    a, b, df, f = SMALL[small](a, b, df, torch.rand((I, J), generator=g, device="cuda"))
    args, plan = [a, b, c.abs(), d], B.Plan(expr)
    split, plain = (evaluate(plan, args, df, n, f=f)[1:] for n in (plan.workspace_bytes, plan.workspace_bytes - 16))
    assert not torch.equal(split[0], plain[0])
    want = exact(args, df, K, f)[1:]
    # (dc is mostly sums beside the products, which are no product's, of other pieces: 5 % either way)
    for s, p, limit in zip(errors(split, want), errors(plain, want), (1.02, 1.02, 1.2)):
        assert s <= limit * p, (s, p)


# tall tiles in short pieces, in long ones with totals in the kernel; low tiles; the most pieces of a size, on the 32-bit kernels alone
@pytest.mark.parametrize("I,J,K,side", [(64, 2048, 32, "a"), (1024, 64, 96, "b"), (8192, 8192, 160, "a"), (8192, 8192, 160, "b"), (512, 8192, 160, "a"), (8192, 512, 256, "b"), (8192, 8192, 32, "a"), (8192, 8192, 96, "b")])
def test_long_sums_of_one_sign(I, J, K, side):
    """da (P, a small) or db (T, b small) of terms of one sign, with the longest sums and the fewest pieces of a size, or with up to 64.  Eight chains of additions of
    two terms round their sums, of up to an eighth of the C terms, C / 16 times each, and seven more times: independent roundings of at most 2^-24,
    2^-24 / sqrt(3) on average, of partial sums that grow evenly, are 2^-24 / sqrt(3) sqrt(C / 384 + 8 / 3) of the result together."""
    import math
    import torch
    from paper_1711_01348_amd import binding as B
    expr, args, df = tensors(I, J, K)
    args, df = [t.abs() for t in args], df.abs()
    args[0 if side == "a" else 1] *= 1e-3
    plan, q, C = B.Plan(expr), 1 if side == "a" else 2, J if side == "a" else I
    g = torch.Generator(device="cuda")
    g.manual_seed(4)
    f = torch.rand((I, J), generator=g, device="cuda")
    want = exact(args, df, K, f)
    # what the other sums beside the products decide: db and dc, or da; the sum of every piece and the result are rounded once, the sums themselves are exact
    beside = (2, 3) if side == "a" else (1,)
    for ws_bytes in {plan.workspace_bytes, plan.workspace_bytes - 16 * (I * J >= 1 << 20)}:   # (small: the family's alone)
        e = errors(evaluate(plan, args, df, ws_bytes, f=f), want)
        assert e[q] <= 2.0 ** -24 / math.sqrt(3) * math.sqrt(C / 384 + 8 / 3)
        assert all(e[n] <= 2.0 ** -24 / math.sqrt(3) * math.sqrt(2) for n in beside), e


@pytest.mark.parametrize("wanted", [(0,), (1,), (2,), (3,), (0, 3), (1, 2)])
def test_any_of_the_gradients(wanted):
    import torch
    from paper_1711_01348_amd import binding as B
    expr, args, df = tensors(1409, 1412, 96)
    plan = B.Plan(expr)
    for ws_bytes in (plan.workspace_bytes, plan.workspace_bytes - 16):
        both = evaluate(plan, args, df, ws_bytes)
        some = evaluate(plan, args, df, ws_bytes, wanted)
        for q, t in zip(wanted, some[1:]):
            # (pieces of the sums depend on which of them are wanted)
            assert ((t.double() - both[1 + q].double()).norm() <= 1e-6 * both[1 + q].double().norm()).item()


# few rows on one side: up to 64 pieces of the other sum, in the room the first one leaves
@pytest.mark.parametrize("I,J,K", [(4096, 64, 32), (64, 4096, 96), (70, 8200, 64), (3000, 132, 288), (33, 68, 32)])
def test_pieces_of_long_sums_for_few_rows(I, J, K):
    from paper_1711_01348_amd import binding as B
    expr, args, df = tensors(I, J, K)
    plan = B.Plan(expr)
    assert plan.forward_family == "worked_mfma"
    for g, w in zip(evaluate(plan, args, df, plan.workspace_bytes), exact(args, df, K)):
        assert check.within(g.cpu().numpy(), w.cpu().numpy(), "f32"), check.errors(g.cpu().numpy(), w.cpu().numpy())


@pytest.mark.parametrize("what", ["inf_df", "nan_df", "huge_df", "large_df", "inf_a", "huge_b"])
@pytest.mark.parametrize("I,J,K", [(2048, 3840, 128), (1409, 1540, 160), (512, 8192, 160)])   # low tiles, tall ones without and with totals
def test_what_is_not_finite_is_left_to_the_32_bit_kernels(I, J, K, what):
    import torch
    from paper_1711_01348_amd import binding as B
    expr, args, df = tensors(I, J, K)
    f = torch.rand_like(df)
    if what.endswith("df"):
        df[I - 1, J - 1] = {"inf": float("inf"), "nan": float("nan"), "huge": 3.4e38, "large": 2.0 ** 110}[what[:-3]]   # (large: times 2^24, not finite)
    else:
        args[0 if what == "inf_a" else 1][5, 127] = float("inf") if what == "inf_a" else 3.4e38
    plan = B.Plan(expr)
    split, plain = (evaluate(plan, args, df, n, f=f) for n in (plan.workspace_bytes, plan.workspace_bytes - 16))
    for s, p in zip(split, plain):
        assert torch.equal(s.isnan(), p.isnan()) and torch.equal(s.isinf(), p.isinf())
        both = s.isfinite()
        # rows with a large number among their terms: the order of the pieces differs, the terms do not
        assert bool(((s[both].double() - p[both].double()).abs() <= 1e-5 * p[both].double().abs() + 2e-5 * p[both].double().pow(2).mean().sqrt()).all())
