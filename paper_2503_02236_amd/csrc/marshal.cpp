// Argument marshalling of the calls that a decode step makes by the hundred: vq_gemv, vq_gemv_batch, vq_gemm, vq_attn_decode and
// vq_kv_quantize from Python objects to the C ABI.  What it does is what the functions of the same names in binding.py do by
// ctypes, object for object, and nothing else: every call reads and checks its arguments anew, nothing is kept.  Calls that
// are not plain -- subclasses, tensors and modes that intercept calls, values that fail a check -- return NotImplemented,
// and binding.py takes them its own way, error messages included.
//
// Why: a 256 x 256 product runs 2.9 us on the GPU, and a call through ctypes takes 8 us of the host.
#include <Python.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/ops/empty.h>
#include <ATen/ops/empty_like.h>
#include <c10/core/impl/LocalDispatchKeySet.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <climits>
#include <vector>

#include "vq_mi355x.h"

namespace {

// Addresses of the entry points in the library that binding.py has loaded, and its classes.
struct Library {
    decltype(&vq_gemv) gemv;
    decltype(&vq_gemv_workspace) gemv_workspace;
    decltype(&vq_gemv_batch) gemv_batch;
    decltype(&vq_gemv_batch_workspace) gemv_batch_workspace;
    decltype(&vq_gemm) gemm;
    decltype(&vq_gemm_workspace) gemm_workspace;
    decltype(&vq_attn_decode) attn_decode;
    decltype(&vq_attn_decode_workspace) attn_decode_workspace;
    decltype(&vq_kv_quantize) kv_quantize;
} lib;
PyObject *weight_type, *kv_type, *pack_type, *error_type;
PyObject *s_N, *s_K, *s_v, *s_code_bits, *s_codes, *s_codebooks, *s_scale, *s_pack, *s_hot_entries, *s_cb_tile;
PyObject *s_B, *s_H, *s_D, *s_T, *s_k_codes, *s_v_codes, *s_k_codebooks, *s_v_codebooks, *s_seq_lens;

struct NotPlain {};   // thrown where binding.py has to take the call

struct Ref {   // a new reference
    PyObject *o;
    Ref(PyObject *object, PyObject *name) : o(PyObject_GetAttr(object, name)) {
        if (!o) {
            PyErr_Clear();
            throw NotPlain();
        }
    }
    ~Ref() { Py_DECREF(o); }
    Ref(const Ref &) = delete;
    Ref &operator=(const Ref &) = delete;
};

int as_int(PyObject *o) {
    if (!PyLong_CheckExact(o)) throw NotPlain();
    const long v = PyLong_AsLong(o);
    if (v == -1 && PyErr_Occurred()) {
        PyErr_Clear();
        throw NotPlain();
    }
    if (v < INT_MIN || v > INT_MAX) throw NotPlain();
    return (int)v;
}
int int_attr(PyObject *object, PyObject *name) {
    Ref r(object, name);
    return as_int(r.o);
}

// A tensor that is nothing but memory on the GPU.
const at::Tensor &tensor(PyObject *o) {
    if (!THPVariable_CheckExact(o)) throw NotPlain();
    const at::Tensor &t = THPVariable_Unpack(o);
    const auto keys = t.key_set();
    if (!t.defined() || !t.is_cuda() || !t.has_storage() || t.layout() != at::kStrided || !t.is_contiguous() || keys.has(c10::DispatchKey::Python) ||
        keys.has(c10::DispatchKey::FuncTorchBatched) || keys.has(c10::DispatchKey::FuncTorchGradWrapper) || keys.has(c10::DispatchKey::Functionalize) ||
        keys.has(c10::DispatchKey::Conjugate) || keys.has(c10::DispatchKey::Negative) || keys.has(c10::DispatchKey::ZeroTensor))
        throw NotPlain();
    return t;
}
void *data(PyObject *o, at::ScalarType type) {
    const at::Tensor &t = tensor(o);
    if (t.scalar_type() != type) throw NotPlain();
    return t.data_ptr();
}

// No mode that would see the allocation of an output.
void no_modes() {
    const auto on = c10::impl::tls_local_dispatch_key_set().included_;
    if (at::impl::PythonTorchFunctionTLS::stack_len() > 0 || on.has(c10::DispatchKey::Python) || on.has(c10::DispatchKey::PythonTLSSnapshot) ||
        on.has(c10::DispatchKey::FuncTorchDynamicLayerFrontMode) || on.has(c10::DispatchKey::Functionalize) || on.has(c10::DispatchKey::Tracer))
        throw NotPlain();
}

// VQWeightDev.desc()
class Weight {
public:
    vq_weight_t d{};
    explicit Weight(PyObject *w) {
        if ((PyObject *)Py_TYPE(w) != weight_type) throw NotPlain();
        d.N = int_attr(w, s_N);
        d.K = int_attr(w, s_K);
        d.v = int_attr(w, s_v);
        d.code_bits = int_attr(w, s_code_bits);
        d.hot_entries = int_attr(w, s_hot_entries);
        {
            Ref t(w, s_cb_tile);
            if (t.o != Py_None) {
                if (!PyTuple_CheckExact(t.o) || PyTuple_GET_SIZE(t.o) != 2) throw NotPlain();
                d.cb_tile_n = as_int(PyTuple_GET_ITEM(t.o, 0));
                d.cb_tile_k = as_int(PyTuple_GET_ITEM(t.o, 1));
            }
        }
        {
            Ref t(w, s_codebooks);
            const at::Tensor &cb = tensor(t.o);
            const int64_t n = cb.dim();
            if (n < 3 || cb.size(n - 3) > INT_MAX || cb.size(n - 2) > INT_MAX) throw NotPlain();
            d.n_codebooks = (int)cb.size(n - 3);
            d.n_entries = (int)cb.size(n - 2);
            d.codebooks = data(t.o, at::kHalf);
        }
        {
            Ref t(w, s_codes);
            if (t.o != Py_None) d.codes = data(t.o, d.code_bits == 16 ? at::kUInt16 : at::kByte);
        }
        {
            Ref t(w, s_scale);
            if (t.o != Py_None) d.scale = data(t.o, at::kHalf);
        }
        Ref p(w, s_pack);
        if (p.o != Py_None) {
            if ((PyObject *)Py_TYPE(p.o) != pack_type) throw NotPlain();
            if (PyObject_GetBuffer(p.o, &pack_, PyBUF_SIMPLE) != 0) {
                PyErr_Clear();
                throw NotPlain();
            }
            held_ = true;
            if (pack_.len != (Py_ssize_t)sizeof(vq_gemv_pack_t)) {
                PyBuffer_Release(&pack_);
                held_ = false;
                throw NotPlain();
            }
            d.gemv_pack = (const vq_gemv_pack_t *)pack_.buf;
        }
    }
    ~Weight() {
        if (held_) PyBuffer_Release(&pack_);
    }
    Weight(const Weight &) = delete;
    Weight &operator=(const Weight &) = delete;

private:
    Py_buffer pack_{};
    bool held_ = false;
};

// VQKVDev.desc()
vq_kv_t cache(PyObject *kv) {
    if ((PyObject *)Py_TYPE(kv) != kv_type) throw NotPlain();
    vq_kv_t d{};
    d.B = int_attr(kv, s_B);
    d.H = int_attr(kv, s_H);
    d.D = int_attr(kv, s_D);
    d.T = int_attr(kv, s_T);
    d.v = int_attr(kv, s_v);
    Ref kc(kv, s_k_codes), vc(kv, s_v_codes), kb(kv, s_k_codebooks), vb(kv, s_v_codebooks), sl(kv, s_seq_lens);
    const at::Tensor &cb = tensor(kb.o);
    if (cb.dim() != 4 || cb.size(1) > INT_MAX || cb.size(2) > INT_MAX) throw NotPlain();
    d.cb_groups = (int)cb.size(1);
    d.n_entries = (int)cb.size(2);
    d.k_codes = data(kc.o, at::kByte);
    d.v_codes = data(vc.o, at::kByte);
    d.k_codebooks = data(kb.o, at::kHalf);
    d.v_codebooks = data(vb.o, at::kHalf);
    if (sl.o != Py_None) d.seq_lens = (const int *)data(sl.o, at::kInt);
    return d;
}

// The caller's workspace, or one of the size asked for.
struct Workspace {
    at::Tensor own;
    void *p = nullptr;
    size_t bytes = 0;
    template <typename Query>
    Workspace(PyObject *ws, const at::Device &device, Query query) {
        if (ws != Py_None) {
            const at::Tensor &t = tensor(ws);
            p = t.data_ptr();
            bytes = (size_t)t.numel() * t.element_size();
            return;
        }
        bytes = query();
        if (bytes == 0) return;
        own = at::empty({(int64_t)bytes}, at::TensorOptions().dtype(at::kByte).device(device));
        p = own.data_ptr();
    }
};

void *stream() { return (void *)c10::hip::getCurrentHIPStream().stream(); }

void check(int status, const char *where) {
    if (status == VQ_OK) return;
    PyObject *e = PyObject_CallFunction(error_type, "is", status, where);
    if (e) {
        PyErr_SetObject(error_type, e);
        Py_DECREF(e);
    }
    throw python_error();
}

// f(): a new reference.  NotPlain becomes NotImplemented, C++ exceptions Python ones.
template <typename F>
PyObject *guarded(F f) {
    HANDLE_TH_ERRORS
    try {
        return f();
    } catch (const NotPlain &) {
        Py_RETURN_NOTIMPLEMENTED;
    }
    END_HANDLE_TH_ERRORS
}

#define VQ_WITHOUT_GIL(status, call)  \
    do {                              \
        Py_BEGIN_ALLOW_THREADS        \
        status = call;                \
        Py_END_ALLOW_THREADS          \
    } while (0)

// (w, x, y or None, ws or None): vq_gemv and vq_gemm
template <typename Call, typename Query>
PyObject *product(PyObject *const *args, Py_ssize_t n, Call call, Query query, const char *where) {
    if (n != 4) throw NotPlain();
    no_modes();
    Weight w(args[0]);
    const at::Tensor &x = tensor(args[1]);
    if (x.scalar_type() != at::kHalf || x.dim() < 1 || x.size(0) > INT_MAX) throw NotPlain();
    const int rows = (int)x.size(0);
    at::Tensor own;
    void *y;
    if (args[2] == Py_None) {
        if (w.d.N < 0) throw NotPlain();
        own = at::empty({(int64_t)rows, (int64_t)w.d.N}, x.options());
        y = own.data_ptr();
    } else {
        y = data(args[2], at::kHalf);
    }
    Workspace ws(args[3], x.device(), [&] { return query(&w.d, rows); });
    const void *xp = x.data_ptr();
    void *s = stream();
    int status;
    VQ_WITHOUT_GIL(status, call(&w.d, xp, rows, y, ws.p, ws.bytes, s));
    check(status, where);
    if (args[2] == Py_None) return THPVariable_Wrap(own);
    Py_INCREF(args[2]);
    return args[2];
}

PyObject *gemv(PyObject *, PyObject *const *args, Py_ssize_t n) {
    return guarded([&] { return product(args, n, lib.gemv, lib.gemv_workspace, "vq_gemv"); });
}

PyObject *gemm(PyObject *, PyObject *const *args, Py_ssize_t n) {
    return guarded([&] { return product(args, n, lib.gemm, lib.gemm_workspace, "vq_gemm"); });
}

// References to what the caller's lists held: another thread may change the lists while a call runs without the interpreter's lock.
struct Held {
    std::vector<PyObject *> all;
    PyObject *add(PyObject *o) {
        all.push_back(o);
        Py_INCREF(o);
        return o;
    }
    ~Held() {
        for (PyObject *o : all) Py_DECREF(o);
    }
};

// (list of w, list of x, list of y or None, ws or None)
PyObject *gemv_batch(PyObject *, PyObject *const *args, Py_ssize_t n) {
    return guarded([&]() -> PyObject * {
        if (n != 4 || !PyList_CheckExact(args[0]) || !PyList_CheckExact(args[1]) || !(args[2] == Py_None || PyList_CheckExact(args[2]))) throw NotPlain();
        no_modes();
        constexpr Py_ssize_t kMost = 16;   // (the entry point takes four)
        const Py_ssize_t count = PyList_GET_SIZE(args[0]);
        if (count < 1 || count > kMost || PyList_GET_SIZE(args[1]) != count || (args[2] != Py_None && PyList_GET_SIZE(args[2]) != count)) throw NotPlain();
        Held held;
        std::vector<std::unique_ptr<Weight>> w;
        const vq_weight_t *wp[kMost];
        const void *xp[kMost];
        void *yp[kMost];
        std::vector<at::Tensor> own;
        for (Py_ssize_t i = 0; i < count; ++i) {
            w.emplace_back(new Weight(held.add(PyList_GET_ITEM(args[0], i))));
            wp[i] = &w.back()->d;
            PyObject *x = held.add(PyList_GET_ITEM(args[1], i));
            xp[i] = data(x, at::kHalf);
            if (args[2] == Py_None) {
                if (wp[i]->N < 0) throw NotPlain();
                own.push_back(at::empty({1, (int64_t)wp[i]->N}, THPVariable_Unpack(x).options()));
                yp[i] = own.back().data_ptr();
            } else {
                yp[i] = data(held.add(PyList_GET_ITEM(args[2], i)), at::kHalf);
            }
        }
        Workspace ws(args[3], THPVariable_Unpack(held.all[1]).device(), [&] { return lib.gemv_batch_workspace(wp, (int)count); });
        void *s = stream();
        int status;
        VQ_WITHOUT_GIL(status, lib.gemv_batch(wp, xp, yp, (int)count, ws.p, ws.bytes, s));
        check(status, "vq_gemv_batch");
        if (args[2] != Py_None) {
            Py_INCREF(args[2]);
            return args[2];
        }
        PyObject *list = PyList_New(count);
        if (!list) throw python_error();
        for (Py_ssize_t i = 0; i < count; ++i) PyList_SET_ITEM(list, i, THPVariable_Wrap(own[i]));
        return list;
    });
}

// (kv, q, sm_scale, out or None, ws or None)
PyObject *attn_decode(PyObject *, PyObject *const *args, Py_ssize_t n) {
    return guarded([&]() -> PyObject * {
        if (n != 5 || !PyFloat_CheckExact(args[2])) throw NotPlain();
        no_modes();
        const vq_kv_t kv = cache(args[0]);
        const at::Tensor &q = tensor(args[1]);
        if (q.scalar_type() != at::kHalf) throw NotPlain();
        const float sm_scale = (float)PyFloat_AS_DOUBLE(args[2]);
        at::Tensor own;
        void *out;
        if (args[3] == Py_None) {
            own = at::empty_like(q);
            out = own.data_ptr();
        } else {
            out = data(args[3], at::kHalf);
        }
        Workspace ws(args[4], q.device(), [&] { return lib.attn_decode_workspace(&kv); });
        const void *qp = q.data_ptr();
        void *s = stream();
        int status;
        VQ_WITHOUT_GIL(status, lib.attn_decode(&kv, qp, sm_scale, out, ws.p, ws.bytes, s));
        check(status, "vq_attn_decode");
        if (args[3] == Py_None) return THPVariable_Wrap(own);
        Py_INCREF(args[3]);
        return args[3];
    });
}

// (kv, k_new, v_new, pos)
PyObject *kv_quantize(PyObject *, PyObject *const *args, Py_ssize_t n) {
    return guarded([&]() -> PyObject * {
        if (n != 4) throw NotPlain();
        no_modes();
        const vq_kv_t kv = cache(args[0]);
        const at::Tensor &k = tensor(args[1]);
        if (k.dim() < 3 || k.size(2) > INT_MAX) throw NotPlain();
        const void *kp = data(args[1], at::kHalf), *vp = data(args[2], at::kHalf);
        const int n_new = (int)k.size(2), pos = as_int(args[3]);
        void *s = stream();
        int status;
        VQ_WITHOUT_GIL(status, lib.kv_quantize(&kv, kp, vp, n_new, pos, s));
        check(status, "vq_kv_quantize");
        Py_RETURN_NONE;
    });
}

// (nine addresses, VQWeightDev, VQKVDev, vq_gemv_pack_t, VQError)
PyObject *init(PyObject *, PyObject *args) {
    unsigned long long a[9];
    if (!PyArg_ParseTuple(args, "(KKKKKKKKK)OOOO", &a[0], &a[1], &a[2], &a[3], &a[4], &a[5], &a[6], &a[7], &a[8], &weight_type, &kv_type, &pack_type, &error_type))
        return nullptr;
    for (PyObject *o : {weight_type, kv_type, pack_type, error_type}) Py_INCREF(o);
    lib.gemv = (decltype(lib.gemv))a[0];
    lib.gemv_workspace = (decltype(lib.gemv_workspace))a[1];
    lib.gemv_batch = (decltype(lib.gemv_batch))a[2];
    lib.gemv_batch_workspace = (decltype(lib.gemv_batch_workspace))a[3];
    lib.gemm = (decltype(lib.gemm))a[4];
    lib.gemm_workspace = (decltype(lib.gemm_workspace))a[5];
    lib.attn_decode = (decltype(lib.attn_decode))a[6];
    lib.attn_decode_workspace = (decltype(lib.attn_decode_workspace))a[7];
    lib.kv_quantize = (decltype(lib.kv_quantize))a[8];
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"init", init, METH_VARARGS, nullptr},
    {"gemv", (PyCFunction)(void (*)(void))gemv, METH_FASTCALL, nullptr},
    {"gemv_batch", (PyCFunction)(void (*)(void))gemv_batch, METH_FASTCALL, nullptr},
    {"gemm", (PyCFunction)(void (*)(void))gemm, METH_FASTCALL, nullptr},
    {"attn_decode", (PyCFunction)(void (*)(void))attn_decode, METH_FASTCALL, nullptr},
    {"kv_quantize", (PyCFunction)(void (*)(void))kv_quantize, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() {
    const struct {
        PyObject **at;
        const char *name;
    } names[] = {{&s_N, "N"}, {&s_K, "K"}, {&s_v, "v"}, {&s_code_bits, "code_bits"}, {&s_codes, "codes"}, {&s_codebooks, "codebooks"}, {&s_scale, "scale"},
                 {&s_pack, "pack"}, {&s_hot_entries, "hot_entries"}, {&s_cb_tile, "cb_tile"}, {&s_B, "B"}, {&s_H, "H"}, {&s_D, "D"}, {&s_T, "T"},
                 {&s_k_codes, "k_codes"}, {&s_v_codes, "v_codes"}, {&s_k_codebooks, "k_codebooks"}, {&s_v_codebooks, "v_codebooks"}, {&s_seq_lens, "seq_lens"}};
    for (const auto &n : names)
        if (!(*n.at = PyUnicode_InternFromString(n.name))) return nullptr;
    PyObject *m = PyModule_Create(&module);
    // binding.py compares this with what it runs under before it calls init
    PyObject *built_for = m ? Py_BuildValue("(snnn)", VQ_BUILT_FOR, (Py_ssize_t)sizeof(vq_weight_t), (Py_ssize_t)sizeof(vq_kv_t), (Py_ssize_t)sizeof(vq_gemv_pack_t)) : nullptr;
    if (!built_for || PyModule_AddObject(m, "built_for", built_for) != 0) {
        Py_XDECREF(built_for);
        Py_XDECREF(m);
        return nullptr;
    }
    return m;
}
