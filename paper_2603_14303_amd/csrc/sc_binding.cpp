// Argument marshalling of the calls that a program makes once per layer and token, in C++: what binding.py's wrappers check and pass on,
// read straight from the tensors.  A call that is anything but ordinary (an output to allocate, a tensor subclass, a layout or a type that
// the wrappers refuse) is left to them: every function returns the library's status, or -1 for "not taken", with nothing done.
//
// Bound by the library's launch.  The wrappers' attribute look-ups and ctypes' conversions (some twenty of each a call) took as long again: host
// time of a decode call with a tail 9.7 us, 6.3 so, of two launches for several query rows 13.3 and 8.6.
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/semanticache.h"

namespace {

constexpr int kNotTaken = -1;

// A tensor argument: `t` is NULL for None.  False: not a plain tensor on the GPU.
inline bool take(PyObject *o, const at::Tensor *&t) {
    t = nullptr;
    if (o == Py_None) return true;
    if (!THPVariable_CheckExact(o)) return false;
    t = &THPVariable_Unpack(o);
    return t->is_cuda();
}
inline bool take_some(PyObject *o, const at::Tensor *&t) { return take(o, t) && t != nullptr; }
inline int code(const at::Tensor &t) {
    switch (t.scalar_type()) {
        case at::kFloat: return SC_F32;
        case at::kBFloat16: return SC_BF16;
        default: return -1;
    }
}
inline void *data(const at::Tensor *t) { return t ? t->data_ptr() : nullptr; }
template <typename T> inline T *data(const at::Tensor *t) { return static_cast<T *>(data(t)); }

inline void *pointer(PyObject *o) { return PyLong_AsVoidPtr(o); }

// The call itself runs without the interpreter lock, as under ctypes.
template <typename F> inline int unlocked(F f) {
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = f();
    Py_END_ALLOW_THREADS
    return status;
}
// A tensor without storage (or anything else that throws) is left to the wrapper, which raises its own error.
template <typename F> PyObject *guarded(F f) {
    int status;
    try {
        status = f();
    } catch (...) {
        status = kNotTaken;
    }
    if (PyErr_Occurred()) {
        if (status != kNotTaken) return nullptr;
        PyErr_Clear();
    }
    return PyLong_FromLong(status);
}

struct Cache {      // Kc, Vc, counts, comp_lens and, if any, Kt, Vt, tail_lens
    const at::Tensor *Kc, *Vc, *counts, *lens, *Kt, *Vt, *tail_lens;
    int kv_code, Hkv, cap, tail_cap;
    bool read(PyObject *const *a, PyObject *const *tail, int64_t d) {
        if (!take_some(a[0], Kc) || !take_some(a[1], Vc) || !take_some(a[2], counts) || !take_some(a[3], lens)) return false;
        if (Kc->dim() != 4 || !Kc->is_contiguous() || !Vc->is_contiguous() || !counts->is_contiguous() || !lens->is_contiguous()) return false;
        kv_code = code(*Kc);
        Hkv = (int)Kc->size(1);
        cap = (int)Kc->size(2);
        tail_cap = 0;
        if (tail[0] == Py_None) {
            Kt = Vt = tail_lens = nullptr;
            return kv_code >= 0;
        }
        if (!take_some(tail[0], Kt) || !take_some(tail[1], Vt) || !take_some(tail[2], tail_lens)) return false;
        if (Kt->dim() != 4 || Kt->sizes() != Vt->sizes() || Kt->scalar_type() != Kc->scalar_type() || Vt->scalar_type() != Kc->scalar_type()) return false;
        if (Kt->size(0) != Kc->size(0) || Kt->size(1) != Kc->size(1) || Kt->size(3) != d) return false;
        tail_cap = (int)Kt->size(2);
        return kv_code >= 0 && Kt->is_contiguous() && Vt->is_contiguous() && tail_lens->is_contiguous();
    }
};

// (mask, seq_lens, offsets, num_chunks, stream)
PyObject *segment(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return guarded([&]() {
        const at::Tensor *mask, *seq_lens, *offsets, *num_chunks;
        if (n != 5 || !take_some(a[0], mask) || !take(a[1], seq_lens) || !take_some(a[2], offsets) || !take_some(a[3], num_chunks)) return kNotTaken;
        if (mask->scalar_type() != at::kByte || mask->dim() != 2 || mask->stride(1) != 1 || offsets->dim() != 2) return kNotTaken;
        void *stream = pointer(a[4]);
        const auto *m = data<const uint8_t>(mask);
        const auto *sl = data<const int32_t>(seq_lens);
        auto *off = data<int32_t>(offsets), *nch = data<int32_t>(num_chunks);
        return unlocked([&]() {
            return (int)sc_segment(m, mask->stride(0), sl, (int)mask->size(0), (int)mask->size(1), off, offsets->stride(0), (int)offsets->size(1), nch, nullptr, 0, stream);
        });
    });
}

// (K, V, offsets, num_chunks, tau, seq_lens, cap, Kc, Vc, counts, comp_lens, cluster_id, base_lens, workspace, bytes, stream)
PyObject *merge(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return guarded([&]() {
        const at::Tensor *K, *V, *offsets, *num_chunks, *seq_lens, *Kc, *Vc, *counts, *lens, *ids, *base;
        if (n != 16 || !take_some(a[0], K) || !take_some(a[1], V) || !take_some(a[2], offsets) || !take(a[3], num_chunks) || !take(a[5], seq_lens)) return kNotTaken;
        if (!take_some(a[7], Kc) || !take_some(a[8], Vc) || !take_some(a[9], counts) || !take_some(a[10], lens) || !take(a[11], ids) || !take(a[12], base))
            return kNotTaken;
        if (K->dim() != 4 || K->sizes() != V->sizes() || K->strides() != V->strides() || K->stride(3) != 1 || K->scalar_type() != V->scalar_type()) return kNotTaken;
        if (!Kc->is_contiguous() || !Vc->is_contiguous() || !counts->is_contiguous() || !lens->is_contiguous()) return kNotTaken;
        const double tau = PyFloat_AsDouble(a[4]);
        const long cap = PyLong_AsLong(a[6]);
        const size_t bytes = PyLong_AsSize_t(a[14]);
        void *w = pointer(a[13]), *stream = pointer(a[15]);
        const int in = code(*K), out = code(*Kc);
        if (PyErr_Occurred() || in < 0 || out < 0 || cap != (int)cap || offsets->dim() < 1) return kNotTaken;
        if (base && (Kc->dim() != 4 || Kc->size(2) != cap || !base->is_contiguous())) return kNotTaken;
        const void *k = data(K), *v = data(V);
        const auto *sl = data<const int32_t>(seq_lens), *off = data<const int32_t>(offsets), *nch = data<const int32_t>(num_chunks), *bl = data<const int32_t>(base);
        void *kc = data(Kc), *vc = data(Vc);
        auto *cnt = data<int32_t>(counts), *cl = data<int32_t>(lens), *cid = data<int32_t>(ids);
        const int B = (int)K->size(0), H = (int)K->size(1), N = (int)K->size(2), d = (int)K->size(3);
        return unlocked([&]() {
            if (base)
                return (int)sc_gsc_merge_append(k, v, (sc_dtype)in, K->stride(0), K->stride(1), K->stride(2), sl, off, offsets->stride(0), nch, B, H, N, d, (float)tau,
                                                kc, vc, (sc_dtype)out, (int)cap, cnt, bl, cl, cid, w, bytes, stream);
            return (int)sc_gsc_merge(k, v, (sc_dtype)in, K->stride(0), K->stride(1), K->stride(2), sl, off, offsets->stride(0), nch, B, H, N, d, (float)tau, kc, vc,
                                     (sc_dtype)out, (int)cap, cnt, cl, cid, w, bytes, stream);
        });
    });
}

// (Q, Kc, Vc, counts, comp_lens, scale, O, lse, Kt, Vt, tail_lens, workspace, bytes, stream)
PyObject *decode(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return guarded([&]() {
        const at::Tensor *Q, *O, *lse;
        Cache c;
        if (n != 14 || !take_some(a[0], Q) || Q->dim() != 3 || !Q->is_contiguous()) return kNotTaken;
        const int B = (int)Q->size(0), Hq = (int)Q->size(1), d = (int)Q->size(2);
        if (!c.read(a + 1, a + 8, d) || !take_some(a[6], O) || !take(a[7], lse)) return kNotTaken;
        const double scale = PyFloat_AsDouble(a[5]);
        const size_t bytes = PyLong_AsSize_t(a[12]);
        void *w = pointer(a[11]), *stream = pointer(a[13]);
        const int qc = code(*Q), oc = code(*O);
        if (PyErr_Occurred() || qc < 0 || oc < 0) return kNotTaken;
        const void *q = data(Q), *kc = data(c.Kc), *vc = data(c.Vc), *kt = data(c.Kt), *vt = data(c.Vt);
        const auto *cnt = data<const int32_t>(c.counts), *cl = data<const int32_t>(c.lens), *tl = data<const int32_t>(c.tail_lens);
        void *o = data(O);
        auto *l = data<float>(lse);
        return unlocked([&]() {
            if (c.Kt)
                return (int)sc_decode_attn_tail(q, (sc_dtype)qc, kc, vc, (sc_dtype)c.kv_code, c.cap, cnt, cl, kt, vt, c.tail_cap, tl, B, Hq, c.Hkv, d, (float)scale, o,
                                                (sc_dtype)oc, l, w, bytes, stream);
            return (int)sc_decode_attn(q, (sc_dtype)qc, kc, vc, (sc_dtype)c.kv_code, c.cap, cnt, cl, B, Hq, c.Hkv, d, (float)scale, o, (sc_dtype)oc, l, w, bytes, stream);
        });
    });
}

// (Q, Kc, Vc, counts, comp_lens, scale, O, lse, Kt, Vt, tail_lens, causal, workspace, bytes, stream)
PyObject *multi(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return guarded([&]() {
        const at::Tensor *Q, *O, *lse;
        Cache c;
        if (n != 15 || !take_some(a[0], Q) || Q->dim() != 4 || !Q->is_contiguous()) return kNotTaken;
        const int nq = (int)Q->size(0), B = (int)Q->size(1), Hq = (int)Q->size(2), d = (int)Q->size(3);
        if (!c.read(a + 1, a + 8, d) || !take_some(a[6], O) || !take(a[7], lse)) return kNotTaken;
        const double scale = PyFloat_AsDouble(a[5]);
        const int causal = PyObject_IsTrue(a[11]);
        const size_t bytes = PyLong_AsSize_t(a[13]);
        void *w = pointer(a[12]), *stream = pointer(a[14]);
        const int qc = code(*Q), oc = code(*O);
        if (PyErr_Occurred() || qc < 0 || oc < 0) return kNotTaken;
        const void *q = data(Q), *kc = data(c.Kc), *vc = data(c.Vc), *kt = data(c.Kt), *vt = data(c.Vt);
        const auto *cnt = data<const int32_t>(c.counts), *cl = data<const int32_t>(c.lens), *tl = data<const int32_t>(c.tail_lens);
        void *o = data(O);
        auto *l = data<float>(lse);
        return unlocked([&]() {
            if (c.Kt)
                return (int)sc_multi_attn_tail(q, (sc_dtype)qc, nq, kc, vc, (sc_dtype)c.kv_code, c.cap, cnt, cl, kt, vt, c.tail_cap, tl, causal, B, Hq, c.Hkv, d,
                                               (float)scale, o, (sc_dtype)oc, l, w, bytes, stream);
            return (int)sc_multi_attn(q, (sc_dtype)qc, nq, kc, vc, (sc_dtype)c.kv_code, c.cap, cnt, cl, B, Hq, c.Hkv, d, (float)scale, o, (sc_dtype)oc, l, w, bytes, stream);
        });
    });
}

PyMethodDef methods[] = {
    {"segment", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(segment)), METH_FASTCALL, nullptr},
    {"merge", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(merge)), METH_FASTCALL, nullptr},
    {"decode", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(decode)), METH_FASTCALL, nullptr},
    {"multi", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(multi)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// torch_version: the torch that the tensors' layout is known from; the loader compares it with the one at hand
PyMODINIT_FUNC PyInit__native() {
    PyObject *m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "torch_version", SC_TORCH_VERSION) < 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
