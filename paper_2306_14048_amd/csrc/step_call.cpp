// The Python call of a generation step: tensor checks and the call of h2o_decode_step in one
// native function, because a small step is as short as the call that starts it.  8 heads x 64 slots,
// binary32, all measured in one process: host time per call 3.5 us, 3.1 of them in here (the launch is
// most of that), 5.7 us with the checks in Python and ctypes; on the GPU 2.8 us from launch to launch in
// a replayed graph.  (A profiler's kernel duration of the same step is 3.6 us, 3.1 at least: its
// begin and end stamps enclose more than the step.)
//
// `decode_step` does the plain case only: exact torch tensors of the cache's device, type
// and shape, contiguous, with storage of their own.  Anything else is left to the caller, which
// says what is wrong or takes the general way, and so is every step where this file is not built; no
// exception leaves it.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>
#include "h2o.h"

namespace {

constexpr const char *SPEC = "paper_2306_14048_amd.step_spec";
constexpr long NOT_PLAIN = 1;                     // (statuses of the library are zero or negative)

// What the four tensors of a step have to be
struct Spec {
    int64_t shape[3];
    c10::ScalarType dtype;
    c10::Device device;
};

bool plain(PyObject *o, const Spec &s, void **p)
{
    if (!THPVariable_CheckExact(o)) return false;
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.defined() || t.scalar_type() != s.dtype || t.layout() != c10::kStrided || !t.has_storage() ||
        t.device() != s.device || t.dim() != 3)
        return false;
    const auto n = t.sizes();
    if (n[0] != s.shape[0] || n[1] != s.shape[1] || n[2] != s.shape[2] || !t.is_contiguous()) return false;
    *p = t.data_ptr();
    return true;
}

void free_spec(PyObject *capsule) { delete static_cast<Spec *>(PyCapsule_GetPointer(capsule, SPEC)); }

// step_spec(memory, batch, heads, head_dim, dtype) -> what decode_step checks against: tensors on
// the device of `memory` (the cache's), of the library's element type `dtype`
PyObject *step_spec(PyObject *, PyObject *args)
{
    PyObject *mem;
    long long b, h, d;
    int dtype;
    if (!PyArg_ParseTuple(args, "OLLLi", &mem, &b, &h, &d, &dtype)) return nullptr;
    if (!THPVariable_Check(mem)) return PyErr_Format(PyExc_TypeError, "memory: expected a tensor");
    const c10::ScalarType st = dtype == H2O_F32 ? c10::kFloat : dtype == H2O_F16 ? c10::kHalf : c10::kBFloat16;
    Spec *s = new (std::nothrow) Spec{{b, h, d}, st, THPVariable_Unpack(mem).device()};
    if (!s) return PyErr_NoMemory();
    PyObject *c = PyCapsule_New(s, SPEC, free_spec);
    if (!c) delete s;
    return c;
}

// decode_step(spec, handle, q, k_new, v_new, out, stream) -> the library's status, or 1 if a tensor
// is not the plain case.  stream: None = the current device's current one, or a raw handle.
PyObject *decode_step(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (n != 7) return PyErr_Format(PyExc_TypeError, "decode_step takes 7 arguments, got %zd", n);
    const Spec *s = static_cast<const Spec *>(PyCapsule_GetPointer(a[0], SPEC));
    if (!s) return nullptr;
    void *p[4], *handle = nullptr, *stream = nullptr;
    try {
        if (!PyLong_Check(a[1])) return PyLong_FromLong(NOT_PLAIN);       // (a closed cache has None)
        handle = PyLong_AsVoidPtr(a[1]);
        if (!handle && PyErr_Occurred()) return nullptr;
        for (int i = 0; i < 4; ++i)
            if (!plain(a[2 + i], *s, &p[i])) return PyLong_FromLong(NOT_PLAIN);
        if (a[6] == Py_None) {
            stream = c10::hip::getCurrentHIPStream().stream();
        } else {
            stream = PyLong_AsVoidPtr(a[6]);
            if (!stream && PyErr_Occurred()) return nullptr;
        }
    } catch (...) {
        PyErr_Clear();
        return PyLong_FromLong(NOT_PLAIN);
    }
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = h2o_decode_step(static_cast<h2o_cache *>(handle), p[0], p[1], p[2], p[3], stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

PyMethodDef methods[] = {
    {"step_spec", step_spec, METH_VARARGS, nullptr},
    {"decode_step", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(decode_step)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_step_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__step_call() { return PyModule_Create(&module); }
