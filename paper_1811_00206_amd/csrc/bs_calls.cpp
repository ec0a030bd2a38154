// _native: the Python calls of binding.py for the usual case, in one native step each: check
// the tensors, take what is needed from torch's allocator, call the C ABI on torch's current
// stream.  (Marshalled in Python and through ctypes a call costs 10 us of host time, twice to
// four times what the small products take on the GPU; here about 4, 2.5 of them the launch.)
//
// Every function returns None for anything it does not handle: a tensor of the wrong kind, an
// argument of another type.  The C ABI has not been called then, and binding.py goes the long
// way, which raises the errors.  Once the C ABI has been called its status stands: it is raised
// as BsError and the call is never tried again (BS_ERR_HIP can come after work was enqueued, and
// a sequence that fails at a later step has already advanced its cell state).
#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <Python.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/bs.h"

namespace {

void* current_stream() { return static_cast<void*>(c10::hip::getCurrentHIPStream().stream()); }

// nullptr unless obj is a tensor on the GPU
const at::Tensor* gpu_tensor(PyObject* obj) {
    if (!THPVariable_Check(obj)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(obj);
    return t.is_cuda() && t.layout() == at::kStrided ? &t : nullptr;
}
const at::Tensor* gpu_tensor(PyObject* obj, at::ScalarType type) {
    const at::Tensor* t = gpu_tensor(obj);
    return t && t->scalar_type() == type && t->is_contiguous() ? t : nullptr;
}
const at::Tensor* gpu_floats(PyObject* obj, int64_t n) {
    const at::Tensor* t = gpu_tensor(obj, at::kFloat);
    return t && t->numel() == n ? t : nullptr;
}

int dtype_code(const at::Tensor& t) {
    return t.scalar_type() == at::kFloat ? BS_F32 : t.scalar_type() == at::kHalf ? BS_F16 : -1;
}

bool int_arg(PyObject* obj, int& v) {
    if (!PyLong_CheckExact(obj)) return false;
    int overflow = 0;
    const long l = PyLong_AsLongAndOverflow(obj, &overflow);
    if (overflow || l < INT32_MIN || l > INT32_MAX) return false;
    v = (int)l;
    return true;
}

// the packed matrix of a call: vals [M, K/bank, k] and offsets of the same shape
struct Packed {
    const at::Tensor *vals, *idx;
    int dtype, bank, k;
    int64_t M, K;
    bool read(PyObject* v, PyObject* i, PyObject* b, at::ScalarType idx_type) {
        vals = gpu_tensor(v);
        idx = gpu_tensor(i, idx_type);
        if (!vals || !idx || !vals->is_contiguous() || vals->dim() != 3 || idx->sizes() != vals->sizes()) return false;
        if (!int_arg(b, bank)) return false;
        dtype = dtype_code(*vals);
        M = vals->size(0);
        K = vals->size(1) * bank;
        k = (int)vals->size(2);
        return dtype >= 0;
    }
    at::Tensor floats(at::IntArrayRef size) const { return at::empty(size, vals->options().dtype(at::kFloat)); }
};

// leading dimension of a 2-D fp32 tensor whose rows are contiguous; -1 if it is not one
int64_t row_pitch(const at::Tensor& t) {
    if (t.scalar_type() != at::kFloat || t.dim() != 2) return -1;
    const int64_t rows = t.size(0), n = t.size(1);
    if (n > 1 && t.stride(1) != 1) return -1;
    const int64_t ld = rows > 1 ? t.stride(0) : std::max<int64_t>(n, 1);
    return ld < n ? -1 : ld;
}

// Gives the interpreter lock up for its lifetime; a destructor, since what runs without it may
// throw: allocations, and tensors of a transform when their address is asked for.
struct WithoutLock {
    PyThreadState* state = PyEval_SaveThread();
    ~WithoutLock() { PyEval_RestoreThread(state); }
};

// the status of `call`, which takes new tensors from torch's allocator and calls the C ABI, all
// without the interpreter lock: a full queue makes a launch wait for the GPU, and an allocation
// may go to the driver
template <typename F>
int enqueue(F&& call) {
    const WithoutLock unlocked;
    return call(current_stream());
}

// raises BsError(status, call), which binding.py has put into this module; nullptr
PyObject* failed(PyObject* self, int status, const char* call) {
    PyObject* type = PyObject_GetAttrString(self, "BsError");
    PyObject* error = type ? PyObject_CallFunction(type, "is", status, call) : nullptr;
    if (error) PyErr_SetObject(type, error);
    Py_XDECREF(error);
    Py_XDECREF(type);
    return nullptr;
}

// the caller's `out` object as the result (it is returned, so it gains a reference) or a new one
PyObject* result(PyObject* out, at::Tensor& t) {
    if (out != Py_None) { Py_INCREF(out); return out; }
    return THPVariable_Wrap(std::move(t));
}

// (vals, idx, bank, x, out, wide) -> y
PyObject* spmv(PyObject* self, PyObject* const* args, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    Packed p;
    if (n != 6) Py_RETURN_NONE;
    const bool wide = args[5] == Py_True;
    if (!p.read(args[0], args[1], args[2], wide ? at::kUInt16 : at::kByte)) Py_RETURN_NONE;
    const at::Tensor* x = gpu_floats(args[3], p.K);
    if (!x) Py_RETURN_NONE;
    at::Tensor y;
    const at::Tensor* out = &y;
    if (args[4] != Py_None && !(out = gpu_floats(args[4], p.M))) Py_RETURN_NONE;
    const int status = enqueue([&](void* st) {
        if (out == &y) y = p.floats({p.M});
        const float* xp = static_cast<const float*>(x->const_data_ptr());
        float* yp = static_cast<float*>(out->mutable_data_ptr());
        const void *v = p.vals->const_data_ptr(), *i = p.idx->const_data_ptr();
        return wide ? bs_spmv_wide(v, static_cast<const uint16_t*>(i), p.dtype, p.M, p.K, p.bank, p.k, xp, yp, st)
                    : bs_spmv(v, static_cast<const uint8_t*>(i), p.dtype, p.M, p.K, p.bank, p.k, xp, yp, st);
    });
    if (status != BS_OK) return failed(self, status, wide ? "bs_spmv_wide" : "bs_spmv");
    return result(args[4], y);
    END_HANDLE_TH_ERRORS
}

// (vals, idx, bank, X, out, workspace, wide) -> Y
PyObject* spmm(PyObject* self, PyObject* const* args, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    Packed p;
    if (n != 7) Py_RETURN_NONE;
    const bool wide = args[6] == Py_True;
    if (!p.read(args[0], args[1], args[2], wide ? at::kUInt16 : at::kByte)) Py_RETURN_NONE;
    const at::Tensor* X = gpu_tensor(args[3]);
    if (!X) Py_RETURN_NONE;
    const int64_t ldx = row_pitch(*X);
    if (ldx < 0 || X->size(0) != p.K) Py_RETURN_NONE;
    const int64_t N = X->size(1);
    at::Tensor y, ws;
    const at::Tensor* out = &y;
    int64_t ldy = std::max<int64_t>(N, 1);
    if (args[4] != Py_None) {
        if (!(out = gpu_tensor(args[4]))) Py_RETURN_NONE;
        ldy = row_pitch(*out);
        if (ldy < 0 || out->size(0) != p.M || out->size(1) != N) Py_RETURN_NONE;
    }
    const size_t need = wide ? bs_spmm_workspace_bytes_wide(p.dtype, p.M, p.K, p.bank, p.k, N)
                             : bs_spmm_workspace_bytes(p.dtype, p.M, p.K, p.bank, p.k, N);
    void* wp = nullptr;
    size_t ws_bytes = 0;
    if (args[5] != Py_None) {
        const at::Tensor* w = gpu_tensor(args[5]);
        if (!w) Py_RETURN_NONE;
        wp = w->mutable_data_ptr();
        ws_bytes = (size_t)w->numel() * w->element_size();
    }
    const int status = enqueue([&](void* st) {
        if (out == &y) y = p.floats({p.M, N});
        if (args[5] == Py_None && need) {
            ws_bytes = need < 16 ? 16 : need;
            ws = at::empty({(int64_t)ws_bytes}, p.vals->options().dtype(at::kByte));
            wp = ws.mutable_data_ptr();
        }
        const float* xp = static_cast<const float*>(X->const_data_ptr());
        float* yp = static_cast<float*>(out->mutable_data_ptr());
        const void *v = p.vals->const_data_ptr(), *i = p.idx->const_data_ptr();
        return wide ? bs_spmm_wide(v, static_cast<const uint16_t*>(i), p.dtype, p.M, p.K, p.bank, p.k, xp, N, ldx, yp,
                                   ldy, wp, ws_bytes, st)
                    : bs_spmm(v, static_cast<const uint8_t*>(i), p.dtype, p.M, p.K, p.bank, p.k, xp, N, ldx, yp, ldy,
                              wp, ws_bytes, st);
    });
    if (status != BS_OK) return failed(self, status, wide ? "bs_spmm_wide" : "bs_spmm");
    return result(args[4], y);
    END_HANDLE_TH_ERRORS
}

// two results as a tuple: the caller's, or new ones
PyObject* pair(PyObject* out, at::Tensor& a, at::Tensor& b) {
    if (out != Py_None) { Py_INCREF(out); return out; }
    PyObject* pa = THPVariable_Wrap(std::move(a));
    PyObject* pb = pa ? THPVariable_Wrap(std::move(b)) : nullptr;
    PyObject* t = pb ? PyTuple_New(2) : nullptr;
    if (!t) { Py_XDECREF(pa); Py_XDECREF(pb); return nullptr; }
    PyTuple_SET_ITEM(t, 0, pa);
    PyTuple_SET_ITEM(t, 1, pb);
    return t;
}

// vals and idx of a result: [M, nb, k] each
struct PackedOut {
    const at::Tensor& like;
    at::ScalarType idx_type;
    int64_t size[3];
    at::Tensor v, i;
    // false unless `out` is None or a tuple of two such tensors
    bool read(PyObject* out) {
        if (out == Py_None) return true;
        if (!PyTuple_CheckExact(out) || PyTuple_GET_SIZE(out) != 2) return false;
        const at::Tensor* tv = gpu_tensor(PyTuple_GET_ITEM(out, 0), like.scalar_type());
        const at::Tensor* ti = gpu_tensor(PyTuple_GET_ITEM(out, 1), idx_type);
        const at::IntArrayRef shape(size, 3);
        if (!tv || !ti || tv->sizes() != shape || ti->sizes() != shape) return false;
        v = *tv;
        i = *ti;
        return true;
    }
    void allocate() {   // unless the caller brought them
        if (v.defined()) return;
        const at::IntArrayRef shape(size, 3);
        v = at::empty(shape, like.options());
        i = at::empty(shape, like.options().dtype(idx_type));
    }
};

// (W, bank, k, out, wide) -> (vals, idx)
PyObject* prune_pack(PyObject* self, PyObject* const* args, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    int bank, k;
    if (n != 5 || !int_arg(args[1], bank) || !int_arg(args[2], k)) Py_RETURN_NONE;
    const at::Tensor* W = gpu_tensor(args[0]);
    if (!W || W->dim() != 2 || !W->is_contiguous()) Py_RETURN_NONE;
    const int dtype = dtype_code(*W);
    const int64_t M = W->size(0), K = W->size(1);
    if (dtype < 0 || bank < 1 || K % bank || k < 1 || k > bank) Py_RETURN_NONE;
    const bool wide = args[4] == Py_True;
    PackedOut o{*W, wide ? at::kUInt16 : at::kByte, {M, K / bank, k}};
    if (!o.read(args[3])) Py_RETURN_NONE;
    const int status = enqueue([&](void* st) {
        o.allocate();
        const void* w = W->const_data_ptr();
        void *vp = o.v.mutable_data_ptr(), *ip = o.i.mutable_data_ptr();
        return wide ? bs_prune_pack_wide(w, dtype, M, K, bank, k, vp, static_cast<uint16_t*>(ip), st)
                    : bs_prune_pack(w, dtype, M, K, bank, k, vp, static_cast<uint8_t*>(ip), st);
    });
    if (status != BS_OK) return failed(self, status, wide ? "bs_prune_pack_wide" : "bs_prune_pack");
    return pair(args[3], o.v, o.i);
    END_HANDLE_TH_ERRORS
}

// (vals, idx, bank, k2, out) -> (vals2, idx2)
PyObject* reprune(PyObject* self, PyObject* const* args, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    Packed p;
    int k2;
    if (n != 5 || !p.read(args[0], args[1], args[2], at::kByte) || !int_arg(args[3], k2) || k2 < 1 || k2 > p.k)
        Py_RETURN_NONE;
    PackedOut o{*p.vals, at::kByte, {p.M, p.vals->size(1), k2}};
    if (!o.read(args[4])) Py_RETURN_NONE;
    const int status = enqueue([&](void* st) {
        o.allocate();
        return bs_reprune(p.vals->const_data_ptr(), static_cast<const uint8_t*>(p.idx->const_data_ptr()), p.dtype, p.M,
                          p.K, p.bank, p.k, k2, o.v.mutable_data_ptr(), static_cast<uint8_t*>(o.i.mutable_data_ptr()), st);
    });
    if (status != BS_OK) return failed(self, status, "bs_reprune");
    return pair(args[4], o.v, o.i);
    END_HANDLE_TH_ERRORS
}

// the gate matrix of an LSTM call: 4H x (I + H)
struct Gates : Packed {
    int64_t H, I;
    bool read(PyObject* const* args) {
        if (!Packed::read(args[0], args[1], args[2], at::kByte) || M % 4) return false;
        H = M / 4;
        I = K - H;
        return I >= 1;
    }
};

// (vals, idx, bank, x, h, bias, c, c_out, h_out) -> (c_out, h_out)
PyObject* lstm_step(PyObject* self, PyObject* const* args, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    Gates g;
    if (n != 9 || !g.read(args)) Py_RETURN_NONE;
    const at::Tensor *x = gpu_floats(args[3], g.I), *h = gpu_floats(args[4], g.H);
    const at::Tensor *bias = gpu_floats(args[5], 4 * g.H), *c = gpu_floats(args[6], g.H);
    if (!x || !h || !bias || !c) Py_RETURN_NONE;
    // outputs the caller brings go the long way
    if (args[7] != Py_None || args[8] != Py_None) Py_RETURN_NONE;
    at::Tensor c_out, h_out;
    const int status = enqueue([&](void* st) {
        c_out = g.floats({g.H});
        h_out = g.floats({g.H});
        return bs_lstm_step(g.vals->const_data_ptr(), static_cast<const uint8_t*>(g.idx->const_data_ptr()), g.dtype,
                            g.H, g.I, g.bank, g.k, static_cast<const float*>(x->const_data_ptr()),
                            static_cast<const float*>(h->const_data_ptr()),
                            static_cast<const float*>(bias->const_data_ptr()),
                            static_cast<const float*>(c->const_data_ptr()),
                            static_cast<float*>(c_out.mutable_data_ptr()),
                            static_cast<float*>(h_out.mutable_data_ptr()), st);
    });
    if (status != BS_OK) return failed(self, status, "bs_lstm_step");
    return pair(Py_None, c_out, h_out);
    END_HANDLE_TH_ERRORS
}

// (vals, idx, bank, X, h0, bias, c, H_all) -> H_all
PyObject* lstm_sequence(PyObject* self, PyObject* const* args, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    Gates g;
    if (n != 8 || !g.read(args)) Py_RETURN_NONE;
    const at::Tensor* X = gpu_tensor(args[3], at::kFloat);
    if (!X || X->dim() != 2 || X->size(1) != g.I) Py_RETURN_NONE;
    const int64_t T = X->size(0);
    const at::Tensor *h0 = gpu_floats(args[4], g.H), *bias = gpu_floats(args[5], 4 * g.H), *c = gpu_floats(args[6], g.H);
    if (!h0 || !bias || !c) Py_RETURN_NONE;
    at::Tensor all;
    const at::Tensor* out = &all;
    if (args[7] != Py_None && (!(out = gpu_tensor(args[7], at::kFloat)) || out->numel() < T * g.H)) Py_RETURN_NONE;
    const int status = enqueue([&](void* st) {
        if (out == &all) all = g.floats({T, g.H});
        return bs_lstm_sequence(g.vals->const_data_ptr(), static_cast<const uint8_t*>(g.idx->const_data_ptr()), g.dtype,
                                g.H, g.I, g.bank, g.k, static_cast<const float*>(X->const_data_ptr()), T,
                                static_cast<const float*>(h0->const_data_ptr()),
                                static_cast<const float*>(bias->const_data_ptr()),
                                static_cast<float*>(c->mutable_data_ptr()),
                                static_cast<float*>(out->mutable_data_ptr()), st);
    });
    if (status != BS_OK) return failed(self, status, "bs_lstm_sequence");
    return result(args[7], all);
    END_HANDLE_TH_ERRORS
}

// () -> torch's current stream as an integer
PyObject* stream(PyObject*, PyObject*) {
    HANDLE_TH_ERRORS
    return PyLong_FromVoidPtr(current_stream());
    END_HANDLE_TH_ERRORS
}

#define BS_FAST(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    BS_FAST(spmv), BS_FAST(spmm), BS_FAST(prune_pack), BS_FAST(reprune), BS_FAST(lstm_step), BS_FAST(lstm_sequence),
    {"stream", stream, METH_NOARGS, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) { return PyModule_Create(&module); }
