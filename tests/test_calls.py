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
