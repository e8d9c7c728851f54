// Argument marshalling of binding.py's hot entry points: torch tensors to device pointers, Python integers and the shape
// structure to the C ABI's arguments.  What ctypes takes for that is a third of a call's host time (us, a forward / backward
// step that launches nothing 1.65 / 2.24, here 0.41 / 0.44), and rings of short blocks last as long as their launches.
//
// Each does what the ctypes call of the same entry point does, with the same conversions: the
// library's function is handed over by its address, the interpreter's lock is given up during the call, and `stream` is
// a function that gives the stream's handle.
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>

namespace {

PyTypeObject* shape_type = nullptr;
PyObject* other_integer = nullptr;          // for what is no Python integer

struct ToStop {};          // a Python error is set

void* pointer(PyObject* o) {
    if (THPVariable_Check(o)) {
        const at::Tensor& t = THPVariable_Unpack(o);
        if (t.is_cuda()) return t.data_ptr();
    }
    PyErr_SetString(PyExc_TypeError, "expected a GPU tensor");
    throw ToStop();
}
// as ctypes converts to c_int32 and c_int64: no floats, whatever has __index__, bits beyond are dropped
uint64_t integer(PyObject* o) {
    PyObject* other = nullptr;
    if (!PyIndex_Check(o)) {
        o = other = PyObject_CallOneArg(other_integer, o);
        if (!o) throw ToStop();
    }
    const unsigned long long v = PyLong_AsUnsignedLongLongMask(o);
    Py_XDECREF(other);
    if (v == (unsigned long long)-1 && PyErr_Occurred()) throw ToStop();
    return v;
}
int32_t int32(PyObject* o) { return (int32_t)(uint32_t)integer(o); }
// asked when the tensors have been looked at
void* stream(PyObject* ask) {
    PyObject* o = PyObject_CallNoArgs(ask);
    if (!o) throw ToStop();
    void* const st = reinterpret_cast<void*>((uintptr_t)PyLong_AsUnsignedLongLongMask(o));
    Py_DECREF(o);
    if (PyErr_Occurred()) throw ToStop();
    return st;
}
void* address(PyObject* o) { return reinterpret_cast<void*>((uintptr_t)integer(o)); }
float real(PyObject* o) {
    const double v = PyFloat_AsDouble(o);
    if (v == -1.0 && PyErr_Occurred()) throw ToStop();
    return (float)v;
}
struct Shape {
    Py_buffer b;
    explicit Shape(PyObject* o) {
        if (!shape_type || !PyObject_TypeCheck(o, shape_type)) {
            PyErr_SetString(PyExc_TypeError, "expected a SaShape");
            throw ToStop();
        }
        if (PyObject_GetBuffer(o, &b, PyBUF_SIMPLE)) throw ToStop();
    }
    ~Shape() { PyBuffer_Release(&b); }
    const void* at() const { return b.buf; }
};

template <typename F>
PyObject* run(F call) {
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = call();
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(status);
}
template <typename F>
PyObject* guarded(Py_ssize_t n, Py_ssize_t want, F body) {
    if (n != want) {
        PyErr_Format(PyExc_TypeError, "%zd arguments expected, %zd given", want, n);
        return nullptr;
    }
    try {
        return body();
    } catch (const ToStop&) {
    } catch (const std::exception& e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
    }
    return nullptr;
}

using I = int32_t;
using P = void*;
using C = const void*;
#define ENTRY(name) PyObject* name(PyObject*, PyObject* const* a, Py_ssize_t n)

// (function address, 2 tensors, shape, stream)
ENTRY(two) {
    return guarded(n, 5, [&] {
        const auto f = reinterpret_cast<int (*)(P, P, C, P)>(address(a[0]));
        P t0 = pointer(a[1]), t1 = pointer(a[2]), st = stream(a[4]);
        const Shape s(a[3]);
        return run([&] { return f(t0, t1, s.at(), st); });
    });
}
// (function address, 3 tensors, shape, stream)
ENTRY(three) {
    return guarded(n, 6, [&] {
        const auto f = reinterpret_cast<int (*)(P, P, P, C, P)>(address(a[0]));
        P t0 = pointer(a[1]), t1 = pointer(a[2]), t2 = pointer(a[3]), st = stream(a[5]);
        const Shape s(a[4]);
        return run([&] { return f(t0, t1, t2, s.at(), st); });
    });
}
// (function address, q, k, v, o, lse, q_dev, kv_dev, N, layout, shape, stream)
ENTRY(step_fwd) {
    return guarded(n, 12, [&] {
        const auto f = reinterpret_cast<int (*)(P, P, P, P, P, I, I, I, I, C, P)>(address(a[0]));
        P t[5];
        for (int i = 0; i < 5; ++i) t[i] = pointer(a[1 + i]);
        const I q = int32(a[6]), kv = int32(a[7]), N = int32(a[8]), layout = int32(a[9]);
        P st = stream(a[11]);
        const Shape s(a[10]);
        return run([&] { return f(t[0], t[1], t[2], t[3], t[4], q, kv, N, layout, s.at(), st); });
    });
}
// (function address, q, k, v, dout, lse, delta, dq, dk, dv, q_dev, kv_dev, N, layout, shape, stream)
ENTRY(step_bwd) {
    return guarded(n, 16, [&] {
        const auto f = reinterpret_cast<int (*)(P, P, P, P, P, P, P, P, P, I, I, I, I, C, P)>(address(a[0]));
        P t[9];
        for (int i = 0; i < 9; ++i) t[i] = pointer(a[1 + i]);
        const I q = int32(a[10]), kv = int32(a[11]), N = int32(a[12]), layout = int32(a[13]);
        P st = stream(a[15]);
        const Shape s(a[14]);
        return run([&] { return f(t[0], t[1], t[2], t[3], t[4], t[5], t[6], t[7], t[8], q, kv, N, layout, s.at(), st); });
    });
}
// (function address, Q, K, V, O, LSE, N, layout, shape, q_dev_only, stream)
ENTRY(ring_fwd) {
    return guarded(n, 11, [&] {
        const auto f = reinterpret_cast<int (*)(P, P, P, P, P, I, I, C, I, P, P)>(address(a[0]));
        P t[5];
        for (int i = 0; i < 5; ++i) t[i] = pointer(a[1 + i]);
        const I N = int32(a[6]), layout = int32(a[7]), only = int32(a[9]);
        P st = stream(a[10]);
        const Shape s(a[8]);
        return run([&] { return f(t[0], t[1], t[2], t[3], t[4], N, layout, s.at(), only, nullptr, st); });
    });
}
// (function address, Q, K, V, dO, O, LSE, delta, dQ, dK, dV, N, layout, shape, q_dev_only, stream)
ENTRY(ring_bwd) {
    return guarded(n, 16, [&] {
        const auto f = reinterpret_cast<int (*)(P, P, P, P, P, P, P, P, P, P, I, I, C, I, P, P)>(address(a[0]));
        P t[10];
        for (int i = 0; i < 10; ++i) t[i] = pointer(a[1 + i]);
        const I N = int32(a[11]), layout = int32(a[12]), only = int32(a[14]);
        P st = stream(a[15]);
        const Shape s(a[13]);
        return run([&] {
            return f(t[0], t[1], t[2], t[3], t[4], t[5], t[6], t[7], t[8], t[9], N, layout, s.at(), only, nullptr, st);
        });
    });
}
// (function address, x, y, pos, pos_stride_b, shape, base, inverse, stream)
ENTRY(rope) {
    return guarded(n, 9, [&] {
        const auto f = reinterpret_cast<int (*)(P, P, P, int64_t, C, float, I, P)>(address(a[0]));
        P x = pointer(a[1]), y = pointer(a[2]), pos = pointer(a[3]), st = stream(a[8]);
        const int64_t stride = (int64_t)integer(a[4]);
        const float base = real(a[6]);
        const I inverse = int32(a[7]);
        const Shape s(a[5]);
        return run([&] { return f(x, y, pos, stride, s.at(), base, inverse, st); });
    });
}
// What a permutation along axis o moves, rows of `inner` bytes: as an index of t's shape, from the end if negative
struct Extent { int64_t outer, rows, inner; };
Extent extent(const at::Tensor& t, PyObject* o) {
    const int64_t dims = t.dim(), axis = PyNumber_AsSsize_t(o, PyExc_IndexError);
    if (axis == -1 && PyErr_Occurred()) throw ToStop();
    if (axis < -dims || axis >= dims) {
        PyErr_SetString(PyExc_IndexError, "tuple index out of range");
        throw ToStop();
    }
    const int64_t at = axis < 0 ? axis + dims : axis;
    Extent e = {1, t.size(at), t.element_size()};
    for (int64_t i = 0; i < at; ++i) e.outer *= t.size(i);
    for (int64_t i = at + 1; i < dims; ++i) e.inner *= t.size(i);
    return e;
}
const at::Tensor& tensor(PyObject* o) {
    if (!THPVariable_Check(o)) pointer(Py_None);
    return THPVariable_Unpack(o);
}
// (tensor, axis): its extent
ENTRY(extent_of) {
    return guarded(n, 2, [&] {
        const Extent e = extent(tensor(a[0]), a[1]);
        return Py_BuildValue("LLL", (long long)e.outer, (long long)e.rows, (long long)e.inner);
    });
}
// (function address, src, dst, N, seq_axis, stream): the tensors' sizes are looked at here.  None: not contiguous with equal
// shape and type
ENTRY(permute) {
    return guarded(n, 6, [&]() -> PyObject* {
        const auto f = reinterpret_cast<int (*)(P, P, int64_t, int64_t, int64_t, I, P)>(address(a[0]));
        const at::Tensor &src = tensor(a[1]), &dst = tensor(a[2]);
        if (!src.is_contiguous() || !dst.is_contiguous() || src.sizes() != dst.sizes() || src.scalar_type() != dst.scalar_type())
            Py_RETURN_NONE;
        const I N = int32(a[3]);
        const Extent e = extent(src, a[4]);
        P s = pointer(a[1]), d = pointer(a[2]), st = stream(a[5]);
        return run([&] { return f(s, d, e.outer, e.rows, e.inner, N, st); });
    });
}
// (the type of a shape, a function that makes an integer of what is none)
ENTRY(set_up) {
    return guarded(n, 2, [&]() -> PyObject* {
        if (!PyType_Check(a[0]) || !PyCallable_Check(a[1])) {
            PyErr_SetString(PyExc_TypeError, "expected a type and a function");
            return nullptr;
        }
        Py_INCREF(a[0]);
        Py_INCREF(a[1]);
        shape_type = reinterpret_cast<PyTypeObject*>(a[0]);
        other_integer = a[1];
        Py_RETURN_NONE;
    });
}

#define FAST(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {FAST(two), FAST(three), FAST(step_fwd), FAST(step_bwd), FAST(ring_fwd), FAST(ring_bwd), FAST(rope),
                         FAST(permute), FAST(extent_of), FAST(set_up), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() { return PyModule_Create(&module); }
