// The calls of the Python binding in native code: what __init__.py checks of plain device tensors, and the library call.
//
// What bounds a small layer is the host: a call that launches one kernel took 5.2 us, 2.5 of them the launch, the rest attribute lookups of
// three tensors, the sizes and the marshalling of a foreign call.  Here a tensor is checked without going through Python objects: the same
// call takes the host 3.3 us.  A pass among others, where the GPU is now the longer side: 14x14x512, one image, forward 5.3 -> 4.3 us, the
// three passes of a layer of 11 thousand outputs 19.3 -> 17.1.
//
// Every function returns the library's status, or None where an argument is anything but what it takes for granted (a descriptor of the
// package's types, tensors and parameters in device memory of the expected type, size and contiguity, a stream whose handle is a
// number, no function mode active): the
// caller then checks argument by argument, raises, or takes the general way.  The library is not linked: bind() hands over its entry points.
#include <Python.h>
#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/dwconv.h"

namespace {

enum Operand { X, Y, W, DW };                // input and its gradient, output and its gradient, filter, filter gradient (fp32)

typedef int (*dims_fn)(const void *, int32_t *, int32_t *);
typedef int (*three_fn)(const void *, const void *, const void *, void *, void *);
typedef int (*three_ws_fn)(const void *, const void *, const void *, void *, void *, size_t, void *);
typedef int (*whole_fn)(const void *, const void *, const void *, const void *, void *, void *, void *, size_t, void *);

struct Entry {
    const char *symbol;                      // of the library
    bool group;                              // takes a dwconv_group_desc
    int operands;
    Operand operand[5];
    bool workspace;
};
constexpr Entry ENTRIES[] = {
    {"dwconv_fwd", false, 3, {X, W, Y}, false},
    {"dwconv_bwd_data", false, 3, {Y, W, X}, false},
    {"dwconv_bwd_filter", false, 3, {X, Y, DW}, true},
    {"dwconv_bwd_filter_noalloc", false, 3, {X, Y, DW}, false},
    {"dwconv_bwd", false, 5, {X, Y, W, X, DW}, true},
    {"gconv_fwd", true, 3, {X, W, Y}, false},
    {"gconv_bwd_data", true, 3, {Y, W, X}, false},
    {"gconv_bwd_filter", true, 3, {X, Y, DW}, true},
};
constexpr int NENTRIES = sizeof ENTRIES / sizeof ENTRIES[0];

// set once by bind(), under the interpreter's lock
void *entry_points[NENTRIES];
dims_fn dims[2];                             // dwconv_out_dims, gconv_out_dims
PyObject *desc_type[2], *tensor_type, *parameter_type;

// wrappers without memory of their own, or whose memory is not theirs to hand out
const c10::DispatchKeySet WRAPPERS({c10::DispatchKey::Python, c10::DispatchKey::FuncTorchBatched, c10::DispatchKey::FuncTorchGradWrapper,
                                    c10::DispatchKey::Functionalize});

const at::Tensor *plain(PyObject *o)
{
    if ((PyObject *)Py_TYPE(o) != tensor_type && (PyObject *)Py_TYPE(o) != parameter_type) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.defined() || !t.is_cuda() || t.layout() != at::kStrided || t.key_set().has_any(WRAPPERS) || !t.has_storage()) return nullptr;
    return &t;
}

struct DescView {                            // a descriptor's bytes while the call lasts
    Py_buffer view = {};
    ~DescView() { if (view.obj) PyBuffer_Release(&view); }
};

template <int E>
PyObject *call(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    HANDLE_TH_ERRORS
    constexpr Entry e = ENTRIES[E];
    if (nargs != 1 + e.operands + e.workspace + 1) {
        PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
        return nullptr;
    }
    if ((PyObject *)Py_TYPE(args[0]) != desc_type[e.group] || at::impl::torch_function_mode_enabled()) Py_RETURN_NONE;
    DescView d;
    if (PyObject_GetBuffer(args[0], &d.view, PyBUF_SIMPLE) != 0) return nullptr;
    if (d.view.len != (Py_ssize_t)(e.group ? sizeof(dwconv_group_desc) : sizeof(dwconv_desc))) Py_RETURN_NONE;
    // a copy: another thread may write to the descriptor while the library reads it
    dwconv_desc dd = {};
    dwconv_group_desc gd = {};
    const void *desc = e.group ? (const void *)&gd : (const void *)&dd;
    memcpy(e.group ? (void *)&gd : (void *)&dd, d.view.buf, d.view.len);
    int32_t ho = 0, wo = 0;
    if (dims[e.group](desc, &ho, &wo) != 0) Py_RETURN_NONE;
    const int64_t N = e.group ? gd.N : dd.N, C = e.group ? gd.C : dd.C, H = e.group ? gd.H : dd.H, V = e.group ? gd.W : dd.W;
    const int64_t K = e.group ? gd.K : dd.K, O = e.group ? gd.O : C * dd.mult, Cg = e.group ? C / gd.groups : 1;
    const int64_t count[4] = {N * C * H * V, N * O * ho * wo, O * Cg * K * K, O * Cg * K * K};
    const at::ScalarType stored = (e.group ? gd.dtype : dd.dtype) == DWCONV_F32 ? at::kFloat : at::kBFloat16;

    void *p[5] = {};
    for (int i = 0; i < e.operands; ++i) {
        const at::Tensor *t = plain(args[1 + i]);
        const Operand what = e.operand[i];
        if (!t || t->scalar_type() != (what == DW ? at::kFloat : stored) || t->numel() != count[what] || !t->is_contiguous()) Py_RETURN_NONE;
        p[i] = t->data_ptr();
    }
    void *ws = nullptr;
    size_t bytes = 0;
    if (e.workspace) {
        const at::Tensor *t = plain(args[1 + e.operands]);
        if (!t) Py_RETURN_NONE;
        ws = t->data_ptr();
        bytes = (size_t)t->numel() * t->itemsize();
    }
    void *stream;
    PyObject *const given = args[nargs - 1];
    if (given == Py_None) stream = c10::hip::getCurrentHIPStream().stream();
    else {
        PyObject *handle = PyObject_GetAttrString(given, "cuda_stream");
        if (!handle) return nullptr;
        bool taken = PyLong_Check(handle);   // (the foreign call also takes None, a c_void_p and what else stands for a pointer)
        stream = taken ? PyLong_AsVoidPtr(handle) : nullptr;
        Py_DECREF(handle);
        if (PyErr_Occurred()) { PyErr_Clear(); taken = false; }
        if (!taken) Py_RETURN_NONE;
    }
    int rc;
    void *const fn = entry_points[E];
    Py_BEGIN_ALLOW_THREADS                   // (the launch may wait for room in the stream's queue)
    if constexpr (e.operands == 5) rc = ((whole_fn)fn)(desc, p[0], p[1], p[2], p[3], p[4], ws, bytes, stream);
    else if constexpr (e.workspace) rc = ((three_ws_fn)fn)(desc, p[0], p[1], p[2], ws, bytes, stream);
    else rc = ((three_fn)fn)(desc, p[0], p[1], p[2], stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
    END_HANDLE_TH_ERRORS
}

// bind(lookup, Desc, GroupDesc, Tensor, Parameter): lookup(symbol) gives the address of one of the library's functions
PyObject *bind(PyObject *, PyObject *args)
{
    PyObject *lookup, *type[4];
    if (!PyArg_ParseTuple(args, "OOOOO", &lookup, &type[0], &type[1], &type[2], &type[3])) return nullptr;
    auto address = [&](const char *symbol) -> void * {
        PyObject *a = PyObject_CallFunction(lookup, "s", symbol);
        void *p = a ? PyLong_AsVoidPtr(a) : nullptr;
        Py_XDECREF(a);
        return p;
    };
    void *found[NENTRIES + 2];
    for (int i = 0; i < NENTRIES + 2; ++i) {
        found[i] = address(i < NENTRIES ? ENTRIES[i].symbol : i == NENTRIES ? "dwconv_out_dims" : "gconv_out_dims");
        if (PyErr_Occurred()) return nullptr;
        if (!found[i]) { PyErr_SetString(PyExc_RuntimeError, "no such function"); return nullptr; }
    }
    for (int i = 0; i < NENTRIES; ++i) entry_points[i] = found[i];
    dims[0] = (dims_fn)found[NENTRIES];
    dims[1] = (dims_fn)found[NENTRIES + 1];
    for (PyObject *t : type) Py_INCREF(t);   // (kept until the process ends)
    desc_type[0] = type[0]; desc_type[1] = type[1]; tensor_type = type[2]; parameter_type = type[3];
    Py_RETURN_NONE;
}

#define CALL(NAME, E) {NAME, (PyCFunction)(void (*)(void))call<E>, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    CALL("fwd", 0), CALL("bwd_data", 1), CALL("bwd_filter", 2), CALL("bwd_filter_noalloc", 3), CALL("bwd", 4),
    CALL("gconv_fwd", 5), CALL("gconv_bwd_data", 6), CALL("gconv_bwd_filter", 7),
    {"bind", bind, METH_VARARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", "checks and library calls of the binding", -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding() { return PyModule_Create(&module); }
