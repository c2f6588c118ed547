"""Calls with torch tensors: the native checks accept what the checks in Python accept, and refuse what they refuse."""
import os
import subprocess
import sys
import threading

import numpy as np
import pytest

from paper_1711_01348_amd import workloads as wl


class _List(list):   # what the native checks leave to those in Python
    pass


def _worked():
    from paper_1711_01348_amd import binding as B
    w = wl.config1()
    return B.Plan(w.expr), w


def test_host_tensors_are_refused_in_words():
    import torch
    from paper_1711_01348_amd import binding as B
    plan, w = _worked()
    args = [torch.from_numpy(a) for a in w.arg_list()]
    f, ws = torch.empty(w.expr.f_shape, dtype=torch.float64), torch.empty(64, dtype=torch.uint8)
    assert B._calls.forward(B._FORWARD, plan._h.value, plan._spec, args, f, ws, 0) is None
    assert B._calls.backward(B._BACKWARD, plan._h.value, plan._spec, args, f, f, [None] * len(args), ws, 0) is None
    with pytest.raises(TypeError):
        B._calls.forward(B._FORWARD, plan._h.value, plan._spec, args, f, ws)
    with pytest.raises(TypeError):
        B._calls.spec(True, (2,), ((2, "3"),))


@pytest.mark.parametrize("missing", ["libtad.so", "_calls.so"])
def test_a_tree_that_is_not_built_says_what_to_run(tmp_path, missing):
    import paper_1711_01348_amd as package
    tree, here = tmp_path / "paper_1711_01348_amd", os.path.dirname(package.__file__)
    tree.mkdir()
    for name in os.listdir(here):
        if name.endswith((".py", ".so")) and name != missing:
            os.symlink(os.path.join(here, name), tree / name)
    run = subprocess.run([sys.executable, "-c", "import paper_1711_01348_amd.binding"], cwd=tmp_path, capture_output=True, text=True,
                         env=dict(os.environ, PYTHONPATH=str(tmp_path)))
    assert run.returncode != 0
    assert f"{missing} is missing: run `python -c 'import __graft_entry__ as g; g.build()'`" in run.stderr


def _layer():
    """tanh(b + x w): b is read by the outer function."""
    from paper_1711_01348_amd import binding as B
    e = wl.dense_layer_expr(40, 33, 50, "f32")
    return B.Plan(e), wl.random_inputs(e, 4, -0.3, 0.3)


def test_the_native_derived_call_leaves_the_rest_to_python():
    """Answered with None before anything is called: host tensors, an operand that is none, one that has no gradient of its own."""
    import torch
    from paper_1711_01348_amd import binding as B
    plan, w = _layer()
    args = [torch.from_numpy(a) for a in w.arg_list()]
    df, ws = torch.from_numpy(w.df), torch.empty(64, dtype=torch.uint8)
    for which, out in ((0, args[0]), (3, args[0]), (-1, args[0])):
        assert B._calls.derived(B._DERIVED, plan._h.value, plan._spec, args, df, which, out, ws, 0) is None
    with pytest.raises(TypeError):
        B._calls.derived(B._DERIVED, plan._h.value, plan._spec, args, df, 0, args[0], ws)


@pytest.mark.gpu
def test_derived_gradients_with_tensors_of_the_callers():
    import torch
    from paper_1711_01348_amd import binding as B
    plan, w = _layer()
    args = [torch.from_numpy(a).cuda() for a in w.arg_list()]
    df = torch.from_numpy(w.df).cuda()
    wide = torch.empty(args[0].shape[0], 2 * args[0].shape[1], device="cuda")
    for p in range(3):
        d = B.DerivedGradient(plan, p)
        ws = torch.empty(max(d.workspace_bytes, 1), dtype=torch.uint8, device="cuda")
        want = d.evaluate(args, df)
        out = torch.full_like(args[p], float("nan"))
        assert d.evaluate(args, df, out=out, ws=ws) is out
        assert torch.equal(out, want)
        assert torch.equal(d.evaluate(_List(args), df, out=torch.empty_like(out), ws=ws), want)
        kept = out.clone()
        for bad in (out.double(), out.cpu(), out.reshape(-1, 1) if out.dim() == 1 else out.reshape(-1), out[:-1]):
            with pytest.raises(ValueError):
                d.evaluate(args, df, out=bad, ws=ws)
        for bad in (df.double(), df.cpu(), df[:-1], df.t()):
            with pytest.raises(ValueError):
                d.evaluate(args, bad, out=out, ws=ws)
        with pytest.raises(ValueError):
            d.evaluate([wide[:, ::2]] + args[1:], df, out=out, ws=ws)
        assert torch.equal(out, kept)


@pytest.mark.gpu
def test_an_alias_has_no_native_derived_call():
    import torch
    from paper_1711_01348_amd import binding as B
    e = wl.matrix_square_expr(20, "f64")
    plan, w = B.Plan(e), wl.random_inputs(e, 5)
    alias = next(p for p, a in enumerate(e.args) if a.same_as is not None)
    root = e.args[alias].same_as
    args = [torch.from_numpy(a).cuda() if a is not None else None for a in w.arg_list()]
    df = torch.from_numpy(w.df).cuda()
    d = B.DerivedGradient(plan, root)
    out, ws = torch.empty_like(args[root]), torch.empty(max(d.workspace_bytes, 1), dtype=torch.uint8, device="cuda")
    assert B._calls.derived(B._DERIVED, d._h.value, plan._spec, args, df, alias, out, ws, 0) is None
    assert torch.equal(d.evaluate(args, df, out=out, ws=ws), d.evaluate(args, df))


@pytest.mark.gpu
def test_both_ways_of_checking_give_the_same():
    import torch
    plan, w = _worked()
    args = [torch.from_numpy(a).cuda() for a in w.arg_list()]
    df, ws = torch.from_numpy(w.df).cuda(), plan.workspace()
    new = lambda: (torch.empty_like(df), [torch.empty_like(a) for a in args])
    results = []
    for kind in (list, tuple, _List):
        f, grads = new()
        assert plan.forward(kind(args), out=f, ws=ws) is f
        out = kind(grads)
        assert plan.backward(kind(args), f, df, out=out, ws=ws) is out
        results.append([f] + list(grads))
    parameters = [torch.nn.Parameter(a) for a in args]
    f, grads = new()
    plan.forward(parameters, out=f, ws=ws)
    plan.backward(parameters, f, df, out=grads, ws=ws)
    results.append([f] + grads)
    f, grads = new()                                   # one gradient alone
    plan.forward(args, out=f, ws=ws)
    plan.backward(args, f, df, out=[None, grads[1]] + [None] * (len(args) - 2), ws=ws)
    torch.cuda.synchronize()
    for r in results[1:]:
        assert all(torch.equal(x, y) for x, y in zip(r, results[0]))
    assert torch.equal(grads[1], results[0][2])


@pytest.mark.gpu
def test_tensors_that_do_not_fit_are_refused():
    import torch
    plan, w = _worked()
    args = [torch.from_numpy(a).cuda() for a in w.arg_list()]
    df, ws = torch.from_numpy(w.df).cuda(), plan.workspace()
    f, grads = torch.empty_like(df), [torch.empty_like(a) for a in args]
    wide = torch.empty(args[0].shape[0], 2 * args[0].shape[1], dtype=torch.float64, device="cuda")
    for bad in (args[0].float(), args[0][:-1], wide[:, ::2], args[0].cpu(), args[0].reshape(-1)):
        with pytest.raises(ValueError):
            plan.forward([bad] + args[1:], out=f, ws=ws)
        with pytest.raises(ValueError):
            plan.backward(args, f, df, out=[bad] + grads[1:], ws=ws)
    with pytest.raises(ValueError):
        plan.forward(args, out=df.t(), ws=ws)


@pytest.mark.gpu
def test_threads_on_streams_of_their_own():
    import torch
    plan, w = _worked()
    args = [torch.from_numpy(a).cuda() for a in w.arg_list()]
    expected = plan.forward(args)
    torch.cuda.synchronize()
    outs = [None] * 4

    def work(i):
        with torch.cuda.stream(torch.cuda.Stream()):
            f, ws = torch.empty_like(expected), plan.workspace()
            for _ in range(50):
                plan.forward(args, out=f, ws=ws)
            torch.cuda.current_stream().synchronize()
            outs[i] = f.cpu().numpy()

    threads = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert all(np.array_equal(o, expected.cpu().numpy()) for o in outs)
