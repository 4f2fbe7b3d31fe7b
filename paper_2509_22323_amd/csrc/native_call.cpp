// The entry points that launch, called with tensors: checks and marshalling of binding.py in native code.  A call of few tokens
// costs what the host needs to issue it.  us of host time a call by way of ctypes / here, and on the GPU in a graph, H = 2, N = 256,
// D = 64: dense 5.9 / 3.0, 4.2; block-sparse 7.2 / 3.2, 5.6; joint, two segments 11.0 / 3.2, 4.6; selection (two launches) 9.2 / 5.6, 5.0.
//
// Every function returns the library's status, or None for arguments that are not what most calls hand over (subclasses of
// Tensor, tensors without storage, shapes that do not fit, numbers of other types, no workspace): binding.py then goes its own
// way, which has every check and every message.  Nothing is kept from one call for the next.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <limits.h>

#include <torch/csrc/autograd/python_variable.h>

#include "rapid_attn.h"
#include "rapid_cache.h"
#include "rapid_mask.h"

namespace {

PyObject* current_stream = nullptr;                // torch._C._cuda_getCurrentRawStream

decltype(&rapid_attn_dense) attn_dense;
decltype(&rapid_attn_block_sparse) attn_block_sparse;
decltype(&rapid_attn_joint) attn_joint;
decltype(&rapid_attn_joint_select) attn_joint_select;
decltype(&rapid_mask_select) mask_select;
decltype(&rapid_cache_store) cache_store;
decltype(&rapid_cache_reuse) cache_reuse;

// A tensor of exactly that class with memory of its own on a GPU; else null.
const at::Tensor* plain(PyObject* o)
{
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.defined() || !t.has_storage() || t.layout() != at::kStrided || !t.is_cuda()) return nullptr;
    return &t;
}
const at::Tensor* of(PyObject* o, at::ScalarType type)
{
    const at::Tensor* t = plain(o);
    return t && t->scalar_type() == type ? t : nullptr;
}
// Contiguous, on a device, of a type.
const at::Tensor* packed(PyObject* o, at::ScalarType type, int device)
{
    const at::Tensor* t = of(o, type);
    return t && t->is_contiguous() && t->get_device() == device ? t : nullptr;
}

bool integer(PyObject* o, int& v)
{
    if (!PyLong_CheckExact(o)) return false;
    int over = 0;
    const long long x = PyLong_AsLongLongAndOverflow(o, &over);
    if (over || x < INT_MIN || x > INT_MAX) return false;
    v = (int)x;
    return true;
}
bool number(PyObject* o, float& v)
{
    if (PyFloat_CheckExact(o)) { v = (float)PyFloat_AS_DOUBLE(o); return true; }
    int i;
    if (!integer(o, i)) return false;
    v = (float)i;
    return true;
}
bool size(int64_t n, int& v)
{
    if (n < 0 || n > INT_MAX) return false;
    v = (int)n;
    return true;
}

// torch's current stream on the device; false: an exception is set
bool stream_on(int device, void*& stream)
{
    PyObject* d = PyLong_FromLong(device);
    if (!d) return false;
    PyObject* s = PyObject_CallOneArg(current_stream, d);
    Py_DECREF(d);
    if (!s) return false;
    stream = PyLong_AsVoidPtr(s);
    Py_DECREF(s);
    return !(stream == nullptr && PyErr_Occurred());
}

// The call itself, without the interpreter's lock (as ctypes makes it).
template <class Call>
PyObject* launch(int device, Call call)
{
    void* stream;
    if (!stream_on(device, stream)) return nullptr;
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = call(stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(status);
}

// q, k, v, o (or q, k alone) contiguous [B, H, N, D]
struct Bhnd {
    const at::Tensor* t[4];
    int B, H, N, D, device;
};
bool bhnd(PyObject* const* a, int n, Bhnd& x)
{
    for (int i = 0; i < n; ++i) {
        const at::Tensor* t = of(a[i], at::kBFloat16);
        if (!t || t->dim() != 4 || !t->is_contiguous()) return false;
        if (i == 0) {
            x.device = t->get_device();
            if (!size(t->size(0), x.B) || !size(t->size(1), x.H) || !size(t->size(2), x.N) || !size(t->size(3), x.D)) return false;
        } else if (t->sizes() != x.t[0]->sizes() || t->get_device() != x.device) return false;
        x.t[i] = t;
    }
    return true;
}
bool length(PyObject* o, int none, int& v)
{
    if (o == Py_None) { v = none; return true; }
    return integer(o, v);
}
bool is_grid(const at::Tensor& mask, int B, int H, int nb)
{
    return mask.dim() == 4 && mask.size(0) == B && mask.size(1) == H && mask.size(2) == nb && mask.size(3) == nb;
}

// (q, k, v, o, kv_len, scale)
PyObject* dense(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    Bhnd x;
    int kv_len;
    float scale;
    if (n != 6 || !bhnd(a, 4, x) || !length(a[4], x.N, kv_len) || !number(a[5], scale)) Py_RETURN_NONE;
    void *q = x.t[0]->data_ptr(), *k = x.t[1]->data_ptr(), *v = x.t[2]->data_ptr(), *o = x.t[3]->data_ptr();
    return launch(x.device, [&](void* s) { return attn_dense(q, k, v, o, x.B, x.H, x.N, x.D, kv_len, scale, nullptr, 0, s); });
}

// (q, k, v, o, mask, block, kv_len, scale, workspace)
PyObject* block_sparse(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    Bhnd x;
    int block, kv_len;
    float scale;
    if (n != 9 || !bhnd(a, 4, x) || !integer(a[5], block) || !length(a[6], x.N, kv_len) || !number(a[7], scale)) Py_RETURN_NONE;
    const at::Tensor *mask = packed(a[4], at::kByte, x.device), *ws = plain(a[8]);
    if (!mask || block <= 0 || x.N % block != 0 || !is_grid(*mask, x.B, x.H, x.N / block)) Py_RETURN_NONE;
    if (!ws || !ws->is_contiguous() || ws->get_device() != x.device) Py_RETURN_NONE;
    void *q = x.t[0]->data_ptr(), *k = x.t[1]->data_ptr(), *v = x.t[2]->data_ptr(), *o = x.t[3]->data_ptr();
    const auto* m = (const unsigned char*)mask->data_ptr();
    void* w = ws->data_ptr();
    const size_t bytes = ws->nbytes();
    return launch(x.device, [&](void* s) {
        return attn_block_sparse(q, k, v, o, x.B, x.H, x.N, x.D, block, m, kv_len, scale, w, bytes, s);
    });
}

// (q, k, mask, block, kv_len, text_start, tau, scale, workspace)
PyObject* select(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    Bhnd x;
    int block, kv_len, text_start;
    float tau, scale;
    if (n != 9 || !bhnd(a, 2, x) || !integer(a[3], block) || !length(a[4], x.N, kv_len) || !length(a[5], x.N, text_start)) Py_RETURN_NONE;
    if (!number(a[6], tau) || !number(a[7], scale)) Py_RETURN_NONE;
    const at::Tensor *mask = packed(a[2], at::kByte, x.device), *ws = plain(a[8]);
    if (!mask || block <= 0 || x.N % block != 0 || !is_grid(*mask, x.B, x.H, x.N / block) || !ws) Py_RETURN_NONE;
    void *q = x.t[0]->data_ptr(), *k = x.t[1]->data_ptr(), *w = ws->data_ptr();
    auto* m = (unsigned char*)mask->data_ptr();
    const size_t bytes = ws->nbytes();
    return launch(x.device, [&](void* s) {
        return mask_select(q, k, x.B, x.H, x.N, x.D, block, kv_len, text_start, tau, scale, m, w, bytes, s);
    });
}

// One or two (q, k, v, o) of [B, H, n, D] with strides.
struct Joint {
    rapid_attn_segment seg[2];
    int n, B, H, N, D, device;
};
bool joint_segments(PyObject* list, Joint& x)
{
    if (!PyList_CheckExact(list) && !PyTuple_CheckExact(list)) return false;
    const Py_ssize_t n = PySequence_Fast_GET_SIZE(list);
    if (n != 1 && n != 2) return false;
    x.n = (int)n;
    int64_t tokens = 0;
    for (Py_ssize_t i = 0; i < n; ++i) {
        PyObject* one = PySequence_Fast_GET_ITEM(list, i);
        if ((!PyList_CheckExact(one) && !PyTuple_CheckExact(one)) || PySequence_Fast_GET_SIZE(one) != 4) return false;
        const at::Tensor* t[4];
        for (int j = 0; j < 4; ++j) {
            t[j] = of(PySequence_Fast_GET_ITEM(one, j), at::kBFloat16);
            if (!t[j] || t[j]->dim() != 4 || t[j]->stride(3) != 1) return false;
            if (j > 0 && (t[j]->sizes() != t[0]->sizes() || t[j]->get_device() != t[0]->get_device())) return false;
            if ((j == 1 || j == 2) && t[j]->strides() != t[0]->strides()) return false;
        }
        int B, H, D;
        rapid_attn_segment& g = x.seg[i];
        if (!size(t[0]->size(0), B) || !size(t[0]->size(1), H) || !size(t[0]->size(2), g.n) || !size(t[0]->size(3), D)) return false;
        if (i == 0) { x.B = B; x.H = H; x.D = D; x.device = t[0]->get_device(); }
        else if (B != x.B || H != x.H || D != x.D) return false;
        g.q = t[0]->data_ptr(); g.k = t[1]->data_ptr(); g.v = t[2]->data_ptr(); g.o = t[3]->data_ptr();
        g.in_stride_b = t[0]->stride(0); g.in_stride_h = t[0]->stride(1); g.in_stride_n = t[0]->stride(2);
        g.out_stride_b = t[3]->stride(0); g.out_stride_h = t[3]->stride(1); g.out_stride_n = t[3]->stride(2);
        tokens += g.n;
    }
    return size(tokens, x.N);
}
bool lengths(PyObject* o, const Joint& x, const int*& p)
{
    p = nullptr;
    if (o == Py_None) return true;
    const at::Tensor* t = packed(o, at::kInt, x.device);
    if (!t || t->numel() != x.B) return false;
    p = (const int*)t->data_ptr();
    return true;
}
inline int blocks(int N, int block) { return block > 0 ? (int)(((long long)N + block - 1) / block) : 0; }

// (segments, mask or None, block, kv_len, kv_lens, scale, workspace)
PyObject* joint(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    Joint x;
    int block, kv_len;
    float scale;
    const int* lens;
    if (n != 7 || !joint_segments(a[0], x) || !integer(a[2], block) || !length(a[3], 0, kv_len) || !lengths(a[4], x, lens)) Py_RETURN_NONE;
    if (!number(a[5], scale)) Py_RETURN_NONE;
    const unsigned char* m = nullptr;
    void* w = nullptr;
    size_t bytes = 0;
    if (a[1] != Py_None) {
        const at::Tensor *mask = packed(a[1], at::kByte, x.device), *ws = plain(a[6]);
        if (!mask || !ws || !is_grid(*mask, x.B, x.H, blocks(x.N, block))) Py_RETURN_NONE;
        m = (const unsigned char*)mask->data_ptr();
        w = ws->data_ptr();
        bytes = ws->nbytes();
    }
    return launch(x.device, [&](void* s) {
        return attn_joint(x.seg, x.n, x.B, x.H, x.D, block, m, kv_len, lens, scale, w, bytes, s);
    });
}

// (segments, block, kv_len, kv_lens, text_start, tau, scale, mask_out or None, workspace)
PyObject* joint_select(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    Joint x;
    int block, kv_len, text_start;
    float tau, scale;
    const int* lens;
    if (n != 9 || !joint_segments(a[0], x) || !integer(a[1], block) || !length(a[2], 0, kv_len) || !lengths(a[3], x, lens)) Py_RETURN_NONE;
    if (!length(a[4], x.N, text_start) || !number(a[5], tau) || !number(a[6], scale)) Py_RETURN_NONE;
    const at::Tensor* ws = plain(a[8]);
    if (!ws) Py_RETURN_NONE;
    unsigned char* m = nullptr;
    if (a[7] != Py_None) {
        const at::Tensor* mask = packed(a[7], at::kByte, x.device);
        if (!mask || !is_grid(*mask, x.B, x.H, blocks(x.N, block))) Py_RETURN_NONE;
        m = (unsigned char*)mask->data_ptr();
    }
    void* w = ws->data_ptr();
    const size_t bytes = ws->nbytes();
    return launch(x.device, [&](void* s) {
        return attn_joint_select(x.seg, x.n, x.B, x.H, x.D, block, kv_len, lens, text_start, tau, scale, m, w, bytes, s);
    });
}

// (a, b, out, flags or None)
template <class Call>
PyObject* residual(PyObject* const* a, Py_ssize_t n, Call call)
{
    if (n != 4) Py_RETURN_NONE;
    const at::Tensor* t[3];
    for (int i = 0; i < 3; ++i) {
        t[i] = of(a[i], at::kBFloat16);
        if (!t[i] || !t[i]->is_contiguous() || t[i]->dim() < 1) Py_RETURN_NONE;
        if (i > 0 && (t[i]->sizes() != t[0]->sizes() || t[i]->get_device() != t[0]->get_device())) Py_RETURN_NONE;
    }
    int B;
    if (!size(t[0]->size(0), B)) Py_RETURN_NONE;
    const size_t per = B > 0 ? (size_t)(t[0]->numel() / B) : 0;
    const int device = t[0]->get_device();
    const unsigned char* flags = nullptr;
    if (a[3] != Py_None) {
        const at::Tensor* f = packed(a[3], at::kByte, device);
        if (!f || f->numel() != B) Py_RETURN_NONE;
        flags = (const unsigned char*)f->data_ptr();
    }
    void *x = t[0]->data_ptr(), *y = t[1]->data_ptr(), *out = t[2]->data_ptr();
    return launch(device, [&](void* s) { return call(x, y, out, B, per, flags, s); });
}
PyObject* store(PyObject*, PyObject* const* a, Py_ssize_t n) { return residual(a, n, cache_store); }
PyObject* reuse(PyObject*, PyObject* const* a, Py_ssize_t n) { return residual(a, n, cache_reuse); }

// bind(address of each entry point, ..): of the library that binding.py has loaded
PyObject* bind(PyObject*, PyObject* args)
{
    unsigned long long p[7];
    if (!PyArg_ParseTuple(args, "KKKKKKK", &p[0], &p[1], &p[2], &p[3], &p[4], &p[5], &p[6])) return nullptr;
    attn_dense = (decltype(attn_dense))p[0];
    attn_block_sparse = (decltype(attn_block_sparse))p[1];
    attn_joint = (decltype(attn_joint))p[2];
    attn_joint_select = (decltype(attn_joint_select))p[3];
    mask_select = (decltype(mask_select))p[4];
    cache_store = (decltype(cache_store))p[5];
    cache_reuse = (decltype(cache_reuse))p[6];
    PyObject* c = PyImport_ImportModule("torch._C");
    if (!c) return nullptr;
    Py_XSETREF(current_stream, PyObject_GetAttrString(c, "_cuda_getCurrentRawStream"));
    Py_DECREF(c);
    if (!current_stream) return nullptr;
    Py_RETURN_NONE;
}

// A C++ exception of a tensor's accessor ends as an exception of Python's.
template <PyObject* (*F)(PyObject*, PyObject* const*, Py_ssize_t)>
PyObject* guarded(PyObject* self, PyObject* const* a, Py_ssize_t n)
{
    try {
        return F(self, a, n);
    } catch (const std::exception& e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
}
#define NATIVE(f) {#f, (PyCFunction)(void (*)(void))guarded<f>, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {{"bind", bind, METH_VARARGS, nullptr}, NATIVE(dense), NATIVE(block_sparse), NATIVE(select), NATIVE(joint),
                         NATIVE(joint_select), NATIVE(store), NATIVE(reuse), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "native_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// built_for: the torch and the Python whose headers this was compiled with (binding.py takes no other)
PyMODINIT_FUNC PyInit_native_call(void)
{
    PyObject* m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "built_for", BUILT_FOR) < 0) { Py_DECREF(m); return nullptr; }
    return m;
}
