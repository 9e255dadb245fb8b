// Host path of the Python binding: what happens between a Python call and the C entry point.
//
// A product at the small sizes takes 2-4 us on the GPU, so a call's time is the host's.  Checking the
// arguments, allocating the result, finding the stream and marshalling through ctypes took 6-7 us of
// interpreted code a call; here the same checks read the tensors' fields and the C entry point is called
// through its address.  Python keeps the names, the defaults and the rare paths (lending scratch).
//
// The C library is the one the Python side has loaded: bind() takes its entry points' addresses, so this
// module does not link to it and a process always talks to one library.
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/hip/EmptyTensor.h>
#include <ATen/ops/empty.h>
#include <c10/hip/HIPStream.h>

#include "bsr_spmm.h"

namespace {

bsr_status (*g_spmm)(const bsr_matrix*, int64_t, const void*, void*, bsr_dtype, bsr_path, void*) = nullptr;
bsr_status (*g_spmm_static)(const bsr_matrix*, int64_t, const void*, void*, bsr_dtype, void*) = nullptr;
bsr_status (*g_sddmm)(const bsr_matrix*, int64_t, const void*, const void*, void*, bsr_dtype, void*, size_t, void*) = nullptr;
bsr_status (*g_sddmm_workspace)(const bsr_matrix*, int64_t, size_t*) = nullptr;
bsr_status (*g_scratch_size)(const bsr_matrix*, int64_t, size_t*) = nullptr;
PyObject* g_error = nullptr;                          // BsrError(status, where)

// What the calls need to know of a matrix; owned by the Python object that owns the handle.
struct core_object {
    PyObject_HEAD
    bsr_matrix* handle;
    int64_t n, k, nnzb;
    int64_t bs_r, bs_c;
    int dtype;
    size_t scratch_bytes;                             // what has been lent so far
};

constexpr at::ScalarType kTypes[3] = {at::kFloat, at::kHalf, at::kBFloat16};

int core_init(PyObject* self, PyObject* args, PyObject*)
{
    core_object* c = reinterpret_cast<core_object*>(self);
    unsigned long long handle = 0;
    long long n, k, nnzb, bs_r, bs_c;
    if (!PyArg_ParseTuple(args, "KLLLLLi", &handle, &n, &k, &nnzb, &bs_r, &bs_c, &c->dtype)) return -1;
    c->handle = reinterpret_cast<bsr_matrix*>(handle);
    c->n = n; c->k = k; c->nnzb = nnzb; c->bs_r = bs_r; c->bs_c = bs_c;
    c->scratch_bytes = 0;
    return 0;
}

PyObject* core_lent(PyObject* self, PyObject* bytes)
{
    const size_t v = PyLong_AsSize_t(bytes);
    if (PyErr_Occurred()) return nullptr;
    reinterpret_cast<core_object*>(self)->scratch_bytes = v;
    Py_RETURN_NONE;
}

PyObject* core_closed(PyObject* self, PyObject*)
{
    reinterpret_cast<core_object*>(self)->handle = nullptr;
    Py_RETURN_NONE;
}

PyMethodDef core_methods[] = {
    {"lent", core_lent, METH_O, "The handle has been lent this many bytes of scratch."},
    {"closed", core_closed, METH_NOARGS, "The handle has been destroyed."},
    {nullptr, nullptr, 0, nullptr}};

PyTypeObject core_type = {PyVarObject_HEAD_INIT(nullptr, 0)};

PyObject* value_error(const char* text)
{
    PyErr_SetString(PyExc_ValueError, text);
    return nullptr;
}

// Code of a tensor's type, -1 with KeyError(dtype) for a type the library has not.
int type_code(const at::Tensor& t, PyObject* obj)
{
    const at::ScalarType s = t.scalar_type();
    for (int i = 0; i < 3; ++i)
        if (s == kTypes[i]) return i;
    PyObject* d = PyObject_GetAttrString(obj, "dtype");
    if (d) { PyErr_SetObject(PyExc_KeyError, d); Py_DECREF(d); }
    return -1;
}

// Code of a type's name ("f32" | "f16" | "bf16"; None or "": `fallback`), -1 with KeyError(name).
int name_code(PyObject* name, int fallback)
{
    if (name == Py_None) return fallback;
    if (PyUnicode_Check(name)) {
        Py_ssize_t len = 0;
        const char* s = PyUnicode_AsUTF8AndSize(name, &len);
        if (!s) return -1;
        if (len == 0) return fallback;
        if (!strcmp(s, "f32")) return BSR_F32;
        if (!strcmp(s, "f16")) return BSR_F16;
        if (!strcmp(s, "bf16")) return BSR_BF16;
    }
    PyErr_SetObject(PyExc_KeyError, name);
    return -1;
}

bool tensor_of(PyObject* obj, const char* what, const at::Tensor** out)
{
    if (!THPVariable_Check(obj)) {
        PyErr_Format(PyExc_TypeError, "%s must be a torch.Tensor", what);
        return false;
    }
    *out = &THPVariable_Unpack(obj);
    return true;
}

core_object* core_of(PyObject* obj)
{
    if (Py_TYPE(obj) == &core_type) return reinterpret_cast<core_object*>(obj);
    PyErr_SetString(PyExc_TypeError, "W must be a BsrMatrix");
    return nullptr;
}

PyObject* failed(bsr_status st, const char* where)
{
    PyObject* e = PyObject_CallFunction(g_error, "is", (int)st, where);
    if (e) { PyErr_SetObject(reinterpret_cast<PyObject*>(Py_TYPE(e)), e); Py_DECREF(e); }
    return nullptr;
}

// Scratch the product with m rows wants and the handle has not been lent: W.ensure_scratch(m), in Python.
bool ensure_scratch(PyObject* W, const core_object* c, int64_t m)
{
    size_t need = 0;
    const bsr_status st = g_scratch_size(c->handle, m, &need);
    if (st != BSR_OK) { failed(st, "bsr_scratch_size"); return false; }
    if (need <= c->scratch_bytes) return true;
    PyObject* r = PyObject_CallMethod(W, "ensure_scratch", "L", (long long)m);
    Py_XDECREF(r);
    return r != nullptr;
}

void* stream() { return c10::hip::getCurrentHIPStream().stream(); }

// A result: through torch's dispatcher, so that its modes and its deterministic fill see it.
at::Tensor result(at::IntArrayRef shape, int code, const at::Tensor& like)
{
    return at::empty(shape, at::TensorOptions().dtype(kTypes[code]).device(like.device()));
}

bool dims2(const at::Tensor& t, int64_t rows, int64_t cols)
{
    return t.dim() == 2 && t.size(0) == rows && t.size(1) == cols;
}

// spmm(W, core, X, Y or None, y_dtype or None, path) -> Y
PyObject* spmm(PyObject*, PyObject* const* a, Py_ssize_t nargs)
{
    HANDLE_TH_ERRORS
    if (nargs != 6) return value_error("spmm takes 6 arguments");
    core_object* c = core_of(a[1]);
    const at::Tensor *X = nullptr, *Y = nullptr;
    if (!c || !tensor_of(a[2], "X", &X)) return nullptr;
    if (X->dim() != 2 || X->size(1) != c->k) return value_error("X must be (m, k)");
    const int x_code = type_code(*X, a[2]);
    if (x_code < 0) return nullptr;
    if (x_code != c->dtype || !X->is_contiguous()) return value_error("X must be contiguous and of W's dtype");
    const int64_t m = X->size(0);
    const int y_code = name_code(a[4], c->dtype);
    if (y_code < 0 || !ensure_scratch(a[0], c, m)) return nullptr;
    const long path = PyLong_AsLong(a[5]);
    if (path == -1 && PyErr_Occurred()) return nullptr;
    at::Tensor fresh;
    PyObject* out = a[3];
    if (out == Py_None) {
        fresh = result({m, c->n}, y_code, *X);
        Y = &fresh;
    } else {
        if (!tensor_of(out, "Y", &Y)) return nullptr;
        if (!dims2(*Y, m, c->n) || !Y->is_contiguous() || Y->scalar_type() != kTypes[y_code])
            return value_error("Y must be a contiguous (m, n) tensor of y_dtype");
    }
    const void* xp = X->data_ptr();
    void* yp = Y->data_ptr();
    bsr_status st;
    {
        pybind11::gil_scoped_release no_gil;
        st = g_spmm(c->handle, m, xp, yp, (bsr_dtype)y_code, (bsr_path)path, stream());
    }
    if (st != BSR_OK) return failed(st, "bsr_spmm");
    if (out == Py_None) return THPVariable_Wrap(std::move(fresh));
    Py_INCREF(out);
    return out;
    END_HANDLE_TH_ERRORS
}

// spmm_static(core, X, Y) -> Y
PyObject* spmm_static(PyObject*, PyObject* const* a, Py_ssize_t nargs)
{
    HANDLE_TH_ERRORS
    if (nargs != 3) return value_error("spmm_static takes 3 arguments");
    core_object* c = core_of(a[0]);
    const at::Tensor *X = nullptr, *Y = nullptr;
    if (!c || !tensor_of(a[1], "X", &X) || !tensor_of(a[2], "Y", &Y)) return nullptr;
    const int x_code = type_code(*X, a[1]);
    if (x_code < 0) return nullptr;
    if (X->dim() != 2 || X->size(1) != c->k || x_code != c->dtype || !X->is_contiguous())
        return value_error("X must be a contiguous (m, k) tensor of W's dtype");
    const int64_t m = X->size(0);
    if (!dims2(*Y, m, c->n) || Y->scalar_type() != at::kFloat || !Y->is_contiguous())
        return value_error("Y must be a contiguous (m, n) fp32 tensor");
    const void* xp = X->data_ptr();
    void* yp = Y->data_ptr();
    bsr_status st;
    {
        pybind11::gil_scoped_release no_gil;
        st = g_spmm_static(c->handle, m, xp, yp, BSR_F32, stream());
    }
    if (st != BSR_OK) return failed(st, "bsr_spmm_static");
    Py_INCREF(a[2]);
    return a[2];
    END_HANDLE_TH_ERRORS
}

// sddmm(W, core, G, X, D or None, d_dtype or None, lend_scratch) -> D
PyObject* sddmm(PyObject*, PyObject* const* a, Py_ssize_t nargs)
{
    HANDLE_TH_ERRORS
    if (nargs != 7) return value_error("sddmm takes 7 arguments");
    core_object* c = core_of(a[1]);
    const at::Tensor *G = nullptr, *X = nullptr, *D = nullptr;
    if (!c || !tensor_of(a[2], "G", &G) || !tensor_of(a[3], "X", &X)) return nullptr;
    if (G->dim() != 2 || X->dim() != 2 || G->size(0) != X->size(0) || G->size(1) != c->n || X->size(1) != c->k)
        return value_error("G must be (m, n) and X (m, k)");
    const int g_code = type_code(*G, a[2]);
    if (g_code < 0) return nullptr;
    const int x_code = type_code(*X, a[3]);
    if (x_code < 0) return nullptr;
    if (g_code != c->dtype || x_code != c->dtype || !G->is_contiguous() || !X->is_contiguous())
        return value_error("G and X must be contiguous and of W's dtype");
    const int64_t m = G->size(0);
    const int d_code = name_code(a[5], c->dtype);
    if (d_code < 0) return nullptr;
    const int lend = PyObject_IsTrue(a[6]);
    if (lend < 0 || (lend && !ensure_scratch(a[0], c, m))) return nullptr;
    at::Tensor fresh;
    PyObject* out = a[4];
    if (out == Py_None) {
        fresh = result({c->nnzb, c->bs_r, c->bs_c}, d_code, *G);
        D = &fresh;
    } else {
        if (!tensor_of(out, "D", &D)) return nullptr;
        if (D->dim() != 3 || D->size(0) != c->nnzb || D->size(1) != c->bs_r || D->size(2) != c->bs_c ||
            D->scalar_type() != kTypes[d_code] || !D->is_contiguous())
            return value_error("D must be a contiguous (nnzb, bs_r, bs_c) tensor of d_dtype");
    }
    const void *gp = G->data_ptr(), *xp = X->data_ptr();
    void* dp = D->data_ptr();
    // This call's workspace: from torch's allocator, which hands it on in stream order once the call has returned.  The
    // product runs without it too: a caller that lends nothing gets nothing allocated, and memory that is not there is
    // no error.
    size_t ws_bytes = 0;
    at::Tensor ws;
    if (lend) {
        pybind11::gil_scoped_release no_gil;          // the first one of a pattern builds the product's plan: milliseconds
        if (g_sddmm_workspace(c->handle, m, &ws_bytes) != BSR_OK) ws_bytes = 0;
    }
    if (ws_bytes > 0) {
        try {
            ws = at::Tensor(at::detail::empty_cuda({(int64_t)ws_bytes}, at::kByte, G->device(), std::nullopt));
        } catch (const c10::OutOfMemoryError&) {
            ws_bytes = 0;
        }
    }
    bsr_status st;
    {
        pybind11::gil_scoped_release no_gil;
        st = g_sddmm(c->handle, m, gp, xp, dp, (bsr_dtype)d_code, ws_bytes ? ws.data_ptr() : nullptr, ws_bytes, stream());
    }
    if (st != BSR_OK) return failed(st, "bsr_sddmm");
    if (out == Py_None) return THPVariable_Wrap(std::move(fresh));
    Py_INCREF(out);
    return out;
    END_HANDLE_TH_ERRORS
}

// bind(address of bsr_spmm_ex, bsr_spmm_static, bsr_sddmm_ws, bsr_scratch_size, bsr_sddmm_workspace_size, BsrError)
PyObject* bind(PyObject*, PyObject* args)
{
    unsigned long long f[5];
    PyObject* error = nullptr;
    if (!PyArg_ParseTuple(args, "KKKKKO", &f[0], &f[1], &f[2], &f[3], &f[4], &error)) return nullptr;
    g_spmm = reinterpret_cast<decltype(g_spmm)>(f[0]);
    g_spmm_static = reinterpret_cast<decltype(g_spmm_static)>(f[1]);
    g_sddmm = reinterpret_cast<decltype(g_sddmm)>(f[2]);
    g_scratch_size = reinterpret_cast<decltype(g_scratch_size)>(f[3]);
    g_sddmm_workspace = reinterpret_cast<decltype(g_sddmm_workspace)>(f[4]);
    Py_INCREF(error);
    Py_XDECREF(g_error);
    g_error = error;
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"bind", bind, METH_VARARGS, "Take the C library's entry points and the error class."},
    {"spmm", reinterpret_cast<PyCFunction>(spmm), METH_FASTCALL, "spmm(W, core, X, Y, y_dtype, path) -> Y"},
    {"spmm_static", reinterpret_cast<PyCFunction>(spmm_static), METH_FASTCALL, "spmm_static(core, X, Y) -> Y"},
    {"sddmm", reinterpret_cast<PyCFunction>(sddmm), METH_FASTCALL, "sddmm(W, core, G, X, D, d_dtype, lend) -> D"},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", "Native host path of the binding.", -1, methods};

}  // namespace

PyMODINIT_FUNC PyInit__binding()
{
    core_type.tp_name = "_binding.Core";
    core_type.tp_basicsize = sizeof(core_object);
    core_type.tp_flags = Py_TPFLAGS_DEFAULT;
    core_type.tp_new = PyType_GenericNew;
    core_type.tp_init = core_init;
    core_type.tp_methods = core_methods;
    if (PyType_Ready(&core_type) < 0) return nullptr;
    PyObject* m = PyModule_Create(&module);
    if (!m) return nullptr;
    Py_INCREF(&core_type);
    if (PyModule_AddObject(m, "Core", reinterpret_cast<PyObject*>(&core_type)) < 0) return nullptr;
    return m;
}
