// The calls of a step with torch tensors: what binding.Plan checks of its tensors, and the call into libtad.so, in one native function each.
//
// A pass of two short kernels is bound by the host.  In Python a tensor's shape, type, place, layout and address are five calls of 60 to
// 100 ns: 8 x 6 x 5 in 64 bits, 13 tensors and three launches, 16.3 us a pass with the checks in Python, 9.5 here (9.1 of them the two calls
// into libtad.so).
//
// Anything out of the ordinary (another number of operands, a subclass, a tensor that does not fit, an address that torch refuses) is answered with
// None: the caller then takes the checks in Python, which say what is wrong.
#include <Python.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>
#include <vector>

namespace {

constexpr int kMaxArgs = 6;

struct Spec {
    at::ScalarType dtype;
    std::vector<int64_t> f_shape;
    std::vector<std::vector<int64_t>> operands;
    std::vector<char> alias;   // reads the tensor of an earlier operand: has no address of its own
};

using Forward = int (*)(const void *, const void *const *, void *, void *, size_t, void *);
using Backward = int (*)(const void *, const void *const *, const void *, const void *, void *const *, void *, size_t, void *);
using Derived = int (*)(void *, const void *const *, const void *, void *, void *, size_t, void *);

bool read_shape(PyObject *o, std::vector<int64_t> &shape) {
    if (!PyTuple_Check(o)) return false;
    for (Py_ssize_t d = 0; d < PyTuple_GET_SIZE(o); ++d) {
        shape.push_back(PyLong_AsLongLong(PyTuple_GET_ITEM(o, d)));
        if (shape.back() == -1 && PyErr_Occurred()) return false;
    }
    return true;
}

void free_spec(PyObject *c) { delete static_cast<Spec *>(PyCapsule_GetPointer(c, "tad.spec")); }

// spec(is 64 bits, shape of f, (shape or None, ...))
PyObject *make_spec(PyObject *, PyObject *const *args, Py_ssize_t n) {
    if (n != 3 || !PyTuple_Check(args[2])) {
        PyErr_SetString(PyExc_TypeError, "spec(wide, f_shape, operands)");
        return nullptr;
    }
    auto *s = new Spec;
    s->dtype = PyObject_IsTrue(args[0]) ? at::kDouble : at::kFloat;
    bool good = read_shape(args[1], s->f_shape);
    for (Py_ssize_t p = 0; good && p < PyTuple_GET_SIZE(args[2]); ++p) {
        PyObject *o = PyTuple_GET_ITEM(args[2], p);
        s->alias.push_back(o == Py_None);
        s->operands.emplace_back();
        if (o != Py_None) good = read_shape(o, s->operands.back());
    }
    if (good && s->operands.size() <= (size_t)kMaxArgs)
        return PyCapsule_New(s, "tad.spec", free_spec);
    delete s;
    if (!PyErr_Occurred()) PyErr_SetString(PyExc_TypeError, "shapes are tuples of numbers");
    return nullptr;
}

// address of a dense tensor of this type and shape on a GPU, or null
void *address(PyObject *o, const Spec &s, const std::vector<int64_t> &shape) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.is_cuda() || t.scalar_type() != s.dtype || t.dim() != (int64_t)shape.size()) return nullptr;
    const auto sizes = t.sizes();
    for (size_t d = 0; d < shape.size(); ++d)
        if (sizes[d] != shape[d]) return nullptr;
    return t.is_contiguous() ? t.data_ptr() : nullptr;
}

struct Items {   // of a list or tuple
    PyObject *const *at = nullptr;
    Py_ssize_t n = -1;
    explicit Items(PyObject *o) {
        if (PyList_CheckExact(o) || PyTuple_CheckExact(o)) {
            at = PySequence_Fast_ITEMS(o);
            n = PySequence_Fast_GET_SIZE(o);
        }
    }
};

bool operands(PyObject *o, const Spec &s, const void **ptr) {
    const Items args(o);
    if (args.n != (Py_ssize_t)s.operands.size()) return false;
    for (Py_ssize_t p = 0; p < args.n; ++p) {
        ptr[p] = nullptr;
        if (s.alias[p]) continue;
        if (!(ptr[p] = address(args.at[p], s, s.operands[p]))) return false;
    }
    return true;
}

struct Workspace {
    void *p = nullptr;
    size_t n = 0;
    bool good = false;
    explicit Workspace(PyObject *o) {
        if (!THPVariable_CheckExact(o)) return;
        const at::Tensor &t = THPVariable_Unpack(o);
        p = t.data_ptr();
        n = (size_t)t.numel();
        good = true;
    }
};

void *pointer(PyObject *o) { return PyLong_AsVoidPtr(o); }   // (null and an error for what is no number)

const Spec *spec_of(PyObject *o) { return static_cast<const Spec *>(PyCapsule_GetPointer(o, "tad.spec")); }

template <typename F> PyObject *guarded(F body) {
    try {
        return body();
    } catch (...) {   // a tensor without an address: Python says it in torch's words
        Py_RETURN_NONE;
    }
}

// forward(function, plan, spec, operands, f, workspace, stream) -> status, or None
PyObject *forward(PyObject *, PyObject *const *a, Py_ssize_t n) {
    if (n != 7) return PyErr_SetString(PyExc_TypeError, "forward: seven arguments"), nullptr;
    return guarded([&]() -> PyObject * {
        const auto fn = reinterpret_cast<Forward>(pointer(a[0]));
        void *const plan = pointer(a[1]), *const stream = pointer(a[6]);
        const Spec *s = spec_of(a[2]);
        if (!s || PyErr_Occurred()) return nullptr;
        const void *ptr[kMaxArgs];
        if (!operands(a[3], *s, ptr)) Py_RETURN_NONE;
        void *const f = address(a[4], *s, s->f_shape);
        const Workspace ws(a[5]);
        if (!f || !ws.good) Py_RETURN_NONE;
        int rc;
        Py_BEGIN_ALLOW_THREADS
        rc = fn(plan, ptr, f, ws.p, ws.n, stream);
        Py_END_ALLOW_THREADS
        return PyLong_FromLong(rc);
    });
}

// backward(function, plan, spec, operands, f, df, gradients, workspace, stream) -> status, or None
PyObject *backward(PyObject *, PyObject *const *a, Py_ssize_t n) {
    if (n != 9) return PyErr_SetString(PyExc_TypeError, "backward: nine arguments"), nullptr;
    return guarded([&]() -> PyObject * {
        const auto fn = reinterpret_cast<Backward>(pointer(a[0]));
        void *const plan = pointer(a[1]), *const stream = pointer(a[8]);
        const Spec *s = spec_of(a[2]);
        if (!s || PyErr_Occurred()) return nullptr;
        const void *ptr[kMaxArgs];
        void *dptr[kMaxArgs];
        if (!operands(a[3], *s, ptr)) Py_RETURN_NONE;
        void *const f = address(a[4], *s, s->f_shape), *const df = address(a[5], *s, s->f_shape);
        if (!f || !df) Py_RETURN_NONE;
        const Items out(a[6]);
        if (out.n != (Py_ssize_t)s->operands.size()) Py_RETURN_NONE;
        for (Py_ssize_t p = 0; p < out.n; ++p) {
            dptr[p] = nullptr;
            if (out.at[p] == Py_None) continue;
            if (s->alias[p] || !(dptr[p] = address(out.at[p], *s, s->operands[p]))) Py_RETURN_NONE;
        }
        const Workspace ws(a[7]);
        if (!ws.good) Py_RETURN_NONE;
        int rc;
        Py_BEGIN_ALLOW_THREADS
        rc = fn(plan, ptr, f, df, dptr, ws.p, ws.n, stream);
        Py_END_ALLOW_THREADS
        return PyLong_FromLong(rc);
    });
}

// derived(function, derived, spec, operands, df, which operand, its gradient, workspace, stream) -> status, or None
PyObject *derived(PyObject *, PyObject *const *a, Py_ssize_t n) {
    if (n != 9) return PyErr_SetString(PyExc_TypeError, "derived: nine arguments"), nullptr;
    return guarded([&]() -> PyObject * {
        const auto fn = reinterpret_cast<Derived>(pointer(a[0]));
        void *const handle = pointer(a[1]), *const stream = pointer(a[8]);
        const Spec *s = spec_of(a[2]);
        const Py_ssize_t which = PyLong_AsSsize_t(a[5]);
        if (!s || PyErr_Occurred()) return nullptr;
        const void *ptr[kMaxArgs];
        if (!operands(a[3], *s, ptr)) Py_RETURN_NONE;
        if (which < 0 || which >= (Py_ssize_t)s->operands.size() || s->alias[which]) Py_RETURN_NONE;
        void *const df = address(a[4], *s, s->f_shape), *const out = address(a[6], *s, s->operands[which]);
        const Workspace ws(a[7]);
        if (!df || !out || !ws.good) Py_RETURN_NONE;
        int rc;
        Py_BEGIN_ALLOW_THREADS
        rc = fn(handle, ptr, df, out, ws.p, ws.n, stream);
        Py_END_ALLOW_THREADS
        return PyLong_FromLong(rc);
    });
}

PyMethodDef methods[] = {
    {"spec", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(make_spec)), METH_FASTCALL, nullptr},
    {"forward", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(forward)), METH_FASTCALL, nullptr},
    {"backward", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(backward)), METH_FASTCALL, nullptr},
    {"derived", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(derived)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__calls() { return PyModule_Create(&module); }
