// The checks and the argument marshalling of the calls a decode step and a small compression are made of, for the Python
// binding.  In Python they take 2.5 us a call, most of it single reads of tensor attributes, and ctypes another 0.8, more
// than the kernels of a small call leave time for: compression and attention of 4 heads of 512 tokens 14.1 us a pass, 11.1 from here.
//
// Every function returns the status of the C entry point, or None where an argument is not what the call takes: the binding then
// goes through its own checks, which say what is wrong.  Nothing is kept from one call to the next.
#include <Python.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/l2kv.h"

namespace {

// Entry points of the loaded library, set once by bind().
decltype(&l2kv_decode_attn) decode_attn_entry = nullptr;
decltype(&l2kv_decode_attn_out) decode_attn_out_entry = nullptr;
decltype(&l2kv_compress) compress_entry = nullptr;
decltype(&l2kv_keep_count) keep_count_entry = nullptr;

// A plain contiguous device tensor, else nullptr.  (Subclasses of torch.Tensor take the way through Python.)
const at::Tensor* device_tensor(PyObject* o) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    return t.is_cuda() && t.is_contiguous() ? &t : nullptr;
}

bool element_type(const at::Tensor& t, l2kv_dtype* dt) {
    const auto s = t.scalar_type();
    *dt = s == at::kFloat ? L2KV_F32 : L2KV_BF16;
    return s == at::kFloat || s == at::kBFloat16;
}

bool number(PyObject* o, double* v) {
    if (!PyFloat_CheckExact(o) && !PyLong_CheckExact(o)) return false;
    *v = PyFloat_AsDouble(o);
    if (*v == -1.0 && PyErr_Occurred()) {
        PyErr_Clear();
        return false;
    }
    return true;
}

bool integer(PyObject* o, int64_t* v) {
    if (!PyLong_CheckExact(o)) return false;
    *v = PyLong_AsLongLong(o);
    if (*v == -1 && PyErr_Occurred()) {
        PyErr_Clear();
        return false;
    }
    return true;
}

// The handle of the stream a call goes to, from the binding's own function: only asked for when the arguments are in order.
bool stream_handle(PyObject* stream, PyObject* handle_of, void** handle) {
    PyObject* const v = PyObject_CallFunctionObjArgs(handle_of, stream, nullptr);
    if (v == nullptr) return false;
    *handle = PyLong_AsVoidPtr(v);
    Py_DECREF(v);
    return !(*handle == nullptr && PyErr_Occurred());
}

template <typename F> PyObject* guarded(F&& f) {
    try {
        return f();
    } catch (const std::exception&) {           // a tensor without memory, for instance
        Py_RETURN_NONE;
    }
}

template <typename F> PyObject* status_of(F&& call) {
    int st;
    Py_BEGIN_ALLOW_THREADS
    st = (int)call();
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(st);
}

// (Q, Kc, Vc, O, workspace, scale, stream, stream's handle)
template <bool kAnyOutput> PyObject* decode(PyObject* const* a, Py_ssize_t n_args) {
    const at::Tensor *t[5];
    double scale;
    if (n_args != 8 || !number(a[5], &scale)) Py_RETURN_NONE;
    for (int i = 0; i < 5; ++i)
        if ((t[i] = device_tensor(a[i])) == nullptr) Py_RETURN_NONE;
    const at::Tensor &Q = *t[0], &Kc = *t[1], &Vc = *t[2], &O = *t[3], &ws = *t[4];
    l2kv_dtype dt, out_dt;
    if (Q.dim() != 3 || Kc.dim() != 4 || !element_type(Q, &dt) || !element_type(O, &out_dt)) Py_RETURN_NONE;
    const int64_t B = Q.size(0), Hq = Q.size(1), D = Q.size(2), Hkv = Kc.size(1), n = Kc.size(2);
    if (Kc.size(0) != B || Kc.size(3) != D || Vc.sizes() != Kc.sizes() || Kc.scalar_type() != Q.scalar_type() ||
        Vc.scalar_type() != Q.scalar_type() || O.numel() != B * Hq * D || (!kAnyOutput && out_dt != L2KV_F32))
        Py_RETURN_NONE;
    if (B > INT32_MAX || Hq > INT32_MAX || Hkv > INT32_MAX || D > INT32_MAX) Py_RETURN_NONE;
    const void *q = Q.data_ptr(), *k = Kc.data_ptr(), *v = Vc.data_ptr();
    void *o = O.data_ptr(), *w = ws.data_ptr(), *s;
    const size_t bytes = ws.nbytes();
    if (!stream_handle(a[6], a[7], &s)) return nullptr;
    return status_of([&] {
        if constexpr (kAnyOutput)
            return decode_attn_out_entry(q, k, v, dt, (int32_t)B, (int32_t)Hq, (int32_t)Hkv, n, (int32_t)D, n * D, (float)scale,
                                         out_dt, o, w, bytes, s);
        else
            return decode_attn_entry(q, k, v, dt, (int32_t)B, (int32_t)Hq, (int32_t)Hkv, n, (int32_t)D, n * D, (float)scale,
                                     static_cast<float*>(o), w, bytes, s);
    });
}

PyObject* decode_attn(PyObject*, PyObject* const* a, Py_ssize_t n) { return guarded([&] { return decode<false>(a, n); }); }
PyObject* decode_attn_out(PyObject*, PyObject* const* a, Py_ssize_t n) { return guarded([&] { return decode<true>(a, n); }); }

// (K, V, norms, kept_idx, Kc, Vc, workspace, keep_ratio, slab_heads, stream, stream's handle)
PyObject* compress_checked(PyObject* const* a, Py_ssize_t n_args) {
    const at::Tensor *t[7];
    double ratio;
    int64_t slab;
    if (n_args != 11 || !number(a[7], &ratio) || !integer(a[8], &slab)) Py_RETURN_NONE;
    for (int i = 0; i < 7; ++i)
        if ((t[i] = device_tensor(a[i])) == nullptr) Py_RETURN_NONE;
    const at::Tensor &K = *t[0], &V = *t[1], &norms = *t[2], &idx = *t[3], &Kc = *t[4], &Vc = *t[5], &ws = *t[6];
    l2kv_dtype dt;
    if (K.dim() < 2 || idx.dim() < 1 || !element_type(K, &dt)) Py_RETURN_NONE;
    const int64_t T = K.size(-2), D = K.size(-1), k = idx.size(-1);
    int64_t n = 1;
    for (int64_t i = 0; i < K.dim() - 2; ++i) n *= K.size(i);
    const auto type = K.scalar_type();
    if (V.sizes() != K.sizes() || V.scalar_type() != type || Kc.scalar_type() != type || Vc.scalar_type() != type ||
        norms.scalar_type() != at::kFloat || norms.numel() != n * T || idx.scalar_type() != at::kInt || idx.numel() != n * k ||
        Kc.numel() != n * k * D || Vc.numel() != n * k * D || D > INT32_MAX)
        Py_RETURN_NONE;
    // The kernels write as many rows as the ratio says, head after head.  (0: no ratio, which the entry point refuses.)
    const int64_t kept = keep_count_entry(T, ratio);
    if (kept > 0 && (k < kept || (k > kept && n > 1))) Py_RETURN_NONE;
    const void *kp = K.data_ptr(), *vp = V.data_ptr();
    float* np = static_cast<float*>(norms.data_ptr());
    int32_t* ip = static_cast<int32_t*>(idx.data_ptr());
    void *kc = Kc.data_ptr(), *vc = Vc.data_ptr(), *w = ws.data_ptr(), *s;
    const size_t bytes = ws.nbytes();
    if (!stream_handle(a[9], a[10], &s)) return nullptr;
    return status_of([&] { return compress_entry(kp, vp, dt, n, T, (int32_t)D, T * D, ratio, slab, np, ip, kc, vc, w, bytes, s); });
}

PyObject* compress(PyObject*, PyObject* const* a, Py_ssize_t n) { return guarded([&] { return compress_checked(a, n); }); }

PyObject* bind(PyObject*, PyObject* args) {
    unsigned long long attn, attn_out, comp, count;
    if (!PyArg_ParseTuple(args, "KKKK", &attn, &attn_out, &comp, &count)) return nullptr;
    decode_attn_entry = reinterpret_cast<decltype(decode_attn_entry)>(attn);
    decode_attn_out_entry = reinterpret_cast<decltype(decode_attn_out_entry)>(attn_out);
    compress_entry = reinterpret_cast<decltype(compress_entry)>(comp);
    keep_count_entry = reinterpret_cast<decltype(keep_count_entry)>(count);
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {{"bind", bind, METH_VARARGS, nullptr},
                         {"decode_attn", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(decode_attn)), METH_FASTCALL, nullptr},
                         {"decode_attn_out", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(decode_attn_out)), METH_FASTCALL, nullptr},
                         {"compress", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(compress)), METH_FASTCALL, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "l2kv_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit_l2kv_calls() {
    PyObject* const m = PyModule_Create(&module);
    if (m != nullptr && PyModule_AddStringConstant(m, "torch_version", L2KV_TORCH) != 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
