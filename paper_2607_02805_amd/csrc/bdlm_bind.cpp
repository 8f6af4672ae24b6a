// bdlm_bind.cpp -- native marshalling of torch tensors into the C ABI of libbdlm (Python module
// paper_2607_02805_amd._bind).
//
// Each function takes the arguments of the Python function of the same name (positionally, the
// defaults filled in) and answers
//   NotImplemented  the arguments are not the plain case: the Python code takes the call,
//                   converts what can be converted and raises what there is to raise;
//   an int          the status of the C call, which failed (nothing was enqueued);
//   anything else   what the Python function returns; the work was enqueued.
// The plain case: strided GPU tensors of exactly torch.Tensor or Parameter with the shapes and
// strides that the C ABI reads, outputs given or to be allocated, numpy int64 bookkeeping and
// numpy int32 slots, no tensors that intercept torch calls and no such mode.  Nothing is kept
// from one call to the next.
//
// Why native: a call whose kernels take less than its marshalling is bound by the host.  In a
// loop, an fp32 step of 1 row, 4 heads, 16 tokens took 14.0 us through Python and ctypes and
// takes 4.5 us from here (the launch itself is about 3.5); a step and a commit of 8 rows,
// 24 heads, 32 tokens went from 31.1 to 9.6 us per cycle.
#include <Python.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/ops/empty.h>
#include <ATen/ops/empty_like.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>

#include "bdlm.h"

namespace {

PyObject *g_ndarray = nullptr;   // numpy.ndarray

struct General {};               // thrown where the Python code has to take the call
[[noreturn]] void general() { throw General(); }
void need(bool ok) {
    if (!ok) general();
}

const at::Tensor &tensor(PyObject *o) {
    need(THPVariable_CheckExact(o));
    const at::Tensor &t = THPVariable_Unpack(o);
    need(t.is_cuda() && t.layout() == at::kStrided);
    return t;
}
// The interpreter lock is given up while memory is allocated and work enqueued.
struct Unlocked {
    PyThreadState *s = PyEval_SaveThread();
    ~Unlocked() { PyEval_RestoreThread(s); }
};

template <class T = void>
T *ptr(const at::Tensor &t) { return static_cast<T *>(t.data_ptr()); }

// One set of activations x, dt, B, C and its descriptor.
struct Acts {
    const at::Tensor &x, &dt, &B, &C;
    bdlm_desc_t d;
    Acts(PyObject *px, PyObject *pdt, PyObject *pB, PyObject *pC)
        : x(tensor(px)), dt(tensor(pdt)), B(tensor(pB)), C(tensor(pC)) {
        need(x.dim() == 4 && dt.dim() == 3 && B.dim() == 4 && C.dim() == 4);
        const auto ty = x.scalar_type();
        need(ty == at::kBFloat16 || ty == at::kFloat);
        need(dt.scalar_type() == ty && B.scalar_type() == ty && C.scalar_type() == ty);
        const int64_t b = x.size(0), L = x.size(1), H = x.size(2), G = B.size(2), N = B.size(3);
        need(b * L > 0 && dt.size(0) == b && dt.size(1) == L && dt.size(2) == H);
        need(B.size(0) == b && B.size(1) == L && C.sizes() == B.sizes() && C.strides() == B.strides());
        need(x.stride(3) == 1 && dt.stride(2) == 1 && B.stride(3) == 1);
        d.batch = b;
        d.nheads = H;
        d.headdim = x.size(3);
        d.dstate = N;
        d.ngroups = G;
        d.block_len = L;
        d.in_dtype = ty == at::kBFloat16 ? BDLM_DTYPE_BF16 : BDLM_DTYPE_F32;
        d.reserved = 0;
        for (int i = 0; i < 3; ++i) {
            d.x_stride[i] = x.stride(i);
            d.bc_stride[i] = B.stride(i);
        }
        d.dt_stride[0] = dt.stride(0);
        d.dt_stride[1] = dt.stride(1);
    }
    bool like(const Acts &o) const {
        return x.sizes() == o.x.sizes() && dt.sizes() == o.dt.sizes() && B.sizes() == o.B.sizes() &&
               x.strides() == o.x.strides() && dt.strides() == o.dt.strides() && B.strides() == o.B.strides() &&
               x.scalar_type() == o.x.scalar_type();
    }
};

const float *vec(PyObject *o, int64_t n) {
    const at::Tensor &t = tensor(o);
    need(t.scalar_type() == at::kFloat && t.dim() == 1 && t.size(0) == n && t.is_contiguous());
    return ptr<float>(t);
}
// The state pool; its number of slots.
float *pool(PyObject *o, const bdlm_desc_t &d, int64_t *nslots) {
    const at::Tensor &t = tensor(o);
    need(t.scalar_type() == at::kFloat && t.dim() == 5 && t.is_contiguous());
    need(t.size(1) == d.nheads && t.size(2) == d.dstate / 4 && t.size(3) == BDLM_HEADDIM && t.size(4) == 4);
    *nslots = t.size(0);
    return ptr<float>(t);
}
// A float32 output of exactly `shape`: the given tensor, or a new one for None (where None
// asks for one) and True.
at::Tensor out(PyObject *o, at::IntArrayRef shape, const at::Tensor &like) {
    if (o == Py_None || o == Py_True) {
        const Unlocked u;
        return at::empty(shape, like.options().dtype(at::kFloat));
    }
    const at::Tensor &t = tensor(o);
    need(t.scalar_type() == at::kFloat && t.sizes() == shape && t.is_contiguous());
    return t;
}
// An optional output: None is no output.
at::Tensor opt_out(PyObject *o, at::IntArrayRef shape, const at::Tensor &like) {
    return o == Py_None ? at::Tensor() : out(o, shape, like);
}
float *opt_ptr(const at::Tensor &t) { return t.defined() ? ptr<float>(t) : nullptr; }

// A numpy array's buffer, released at the end of the call.
struct Array {
    Py_buffer v{};
    bool held = false;
    ~Array() {
        if (held) PyBuffer_Release(&v);
    }
    void get(PyObject *o, char f0, char f1, int64_t item, int64_t n, bool write) {
        need(PyObject_TypeCheck(o, reinterpret_cast<PyTypeObject *>(g_ndarray)));
        if (PyObject_GetBuffer(o, &v, PyBUF_C_CONTIGUOUS | PyBUF_FORMAT | (write ? PyBUF_WRITABLE : 0)) != 0) {
            PyErr_Clear();
            general();
        }
        held = true;
        need(v.ndim == 1 && v.itemsize == item && v.shape[0] == n && v.format && v.format[1] == 0 &&
             (v.format[0] == f0 || v.format[0] == f1));
    }
};
struct Slots : Array {
    const int32_t *p = nullptr;
    Slots(PyObject *o, int64_t rows) {
        if (o == Py_None) return;
        get(o, 'i', 'i', 4, rows, false);
        p = static_cast<const int32_t *>(v.buf);
    }
};
struct Books : Array {
    int64_t *p;
    Books(PyObject *o, int64_t nslots) {
        get(o, 'l', 'q', 8, nslots, true);
        p = static_cast<int64_t *>(v.buf);
    }
};
int64_t integer(PyObject *o) {
    need(PyLong_CheckExact(o));
    const long long v = PyLong_AsLongLong(o);
    if (v == -1 && PyErr_Occurred()) {
        PyErr_Clear();
        general();
    }
    return v;
}
void *stream_of(PyObject *o) {
    if (o == Py_None) return c10::hip::getCurrentHIPStream().stream();
    PyObject *h = PyObject_GetAttrString(o, "cuda_stream");
    void *p = h && PyLong_CheckExact(h) ? PyLong_AsVoidPtr(h) : nullptr;
    const bool bad = !h || !PyLong_CheckExact(h) || PyErr_Occurred();
    Py_XDECREF(h);
    if (bad) {
        PyErr_Clear();
        general();
    }
    return p;
}
// A byte workspace of `bytes`: the given contiguous tensor, or a new one.
struct Workspace {
    at::Tensor t;
    void *p = nullptr;
    int64_t bytes = 0;
    Workspace(PyObject *o, int64_t want, const at::Tensor &like) {
        if (o == Py_None) {
            if (want == 0) return;
            const Unlocked u;
            t = at::empty({want}, like.options().dtype(at::kByte));
        } else {
            t = tensor(o);
            need(t.is_contiguous());
        }
        p = t.data_ptr();
        bytes = t.numel() * t.element_size();
    }
};

// Enqueues the work with f and answers its outputs, or its status if it failed.  The outputs
// are wrapped first: once a commit is enqueued nothing may send the call to the Python code.
PyObject *item(const at::Tensor &t) {
    if (!t.defined()) Py_RETURN_NONE;
    return THPVariable_Wrap(t);
}
template <class F>
PyObject *enqueue(PyObject *result, F f) {
    if (!result) general();
    int rc;
    {
        const Unlocked u;
        rc = f();
    }
    if (rc == BDLM_OK) return result;
    Py_DECREF(result);
    return PyLong_FromLong(rc);
}
PyObject *pair(const at::Tensor &a, const at::Tensor &b) {
    PyObject *t = PyTuple_New(2);
    if (!t) general();
    PyTuple_SET_ITEM(t, 0, item(a));
    PyTuple_SET_ITEM(t, 1, item(b));
    return t;
}

template <int NARGS, class F>
PyObject *entry(PyObject *const *a, Py_ssize_t n, F f) {
    if (n != NARGS || at::impl::torch_function_mode_enabled() || c10::impl::TorchDispatchModeTLS::any_modes_set())
        Py_RETURN_NOTIMPLEMENTED;
    try {
        return f(a);
    } catch (const General &) {
        PyErr_Clear();
        Py_RETURN_NOTIMPLEMENTED;
    } catch (...) {   // torch refused something (a tensor without storage, no memory): it says so there
        PyErr_Clear();
        Py_RETURN_NOTIMPLEMENTED;
    }
}

#define BDLM_ENTRY(name, nargs) \
    PyObject *name(PyObject *, PyObject *const *args, Py_ssize_t n) { return entry<nargs>(args, n, [](PyObject *const *a) -> PyObject *
#define BDLM_END ); }

// x dt A B C D D_rev h_pool y slot_idx stream
BDLM_ENTRY(scan_block_step, 11) {
    Acts t(a[0], a[1], a[3], a[4]);
    const bdlm_desc_t &d = t.d;
    const float *A = vec(a[2], d.nheads), *D = vec(a[5], d.nheads), *Dr = vec(a[6], d.nheads);
    int64_t ns;
    const float *h = pool(a[7], d, &ns);
    const Slots sl(a[9], d.batch);
    void *s = stream_of(a[10]);
    const at::Tensor y = out(a[8], {d.batch, d.block_len, d.nheads, BDLM_HEADDIM}, t.x);
    float *yp = ptr<float>(y);
    const void *x = ptr(t.x), *dt = ptr(t.dt), *B = ptr(t.B), *C = ptr(t.C);
    return enqueue(item(y), [&] { return bdlm_scan_block_step(&d, x, dt, A, B, C, D, Dr, h, ns, sl.p, yp, s); });
} BDLM_END

// fwd (x dt A B C D), rev (x dt A B C D_rev), h_pool y slot_idx stream
BDLM_ENTRY(scan_block_step_sep, 16) {
    Acts t(a[0], a[1], a[3], a[4]), r(a[6], a[7], a[9], a[10]);
    need(t.like(r));
    const bdlm_desc_t &d = t.d;
    const float *A = vec(a[2], d.nheads), *D = vec(a[5], d.nheads), *Ar = vec(a[8], d.nheads), *Dr = vec(a[11], d.nheads);
    int64_t ns;
    const float *h = pool(a[12], d, &ns);
    const Slots sl(a[14], d.batch);
    void *s = stream_of(a[15]);
    const at::Tensor y = out(a[13], {d.batch, d.block_len, d.nheads, BDLM_HEADDIM}, t.x);
    float *yp = ptr<float>(y);
    const void *x = ptr(t.x), *dt = ptr(t.dt), *B = ptr(t.B), *C = ptr(t.C);
    const void *x2 = ptr(r.x), *dt2 = ptr(r.dt), *B2 = ptr(r.B), *C2 = ptr(r.C);
    return enqueue(item(y), [&] {
        return bdlm_scan_block_step_sep(&d, x, dt, A, B, C, D, x2, dt2, Ar, B2, C2, Dr, h, ns, sl.p, yp, s);
    });
} BDLM_END

// x dt A B C D D_rev h_pool n_committed n_blocks expected slot_idx y_clean stream
BDLM_ENTRY(commit_boundary, 14) {
    Acts t(a[0], a[1], a[3], a[4]);
    const bdlm_desc_t &d = t.d;
    const float *A = vec(a[2], d.nheads), *D = vec(a[5], d.nheads), *Dr = vec(a[6], d.nheads);
    int64_t ns;
    float *h = pool(a[7], d, &ns);
    Books nc(a[8], ns), nb(a[9], ns);
    const int64_t want = integer(a[10]);
    const Slots sl(a[11], d.batch);
    void *s = stream_of(a[13]);
    const at::Tensor y = opt_out(a[12], {d.batch, d.block_len, d.nheads, BDLM_HEADDIM}, t.x);
    float *yp = opt_ptr(y);
    const void *x = ptr(t.x), *dt = ptr(t.dt), *B = ptr(t.B), *C = ptr(t.C);
    return enqueue(item(y), [&] {
        return bdlm_commit_boundary(&d, x, dt, A, B, C, D, Dr, h, ns, sl.p, nc.p, nb.p, want, yp, s);
    });
} BDLM_END

// clean (x dt B C), next (x dt B C), A D D_rev h_pool n_committed n_blocks expected slot_idx y_clean y_next stream
BDLM_ENTRY(commit_step, 19) {
    Acts t(a[0], a[1], a[2], a[3]), r(a[4], a[5], a[6], a[7]);
    need(t.like(r));
    const bdlm_desc_t &d = t.d;
    const float *A = vec(a[8], d.nheads), *D = vec(a[9], d.nheads), *Dr = vec(a[10], d.nheads);
    int64_t ns;
    float *h = pool(a[11], d, &ns);
    Books nc(a[12], ns), nb(a[13], ns);
    const int64_t want = integer(a[14]);
    const Slots sl(a[15], d.batch);
    void *s = stream_of(a[18]);
    const int64_t shape[4] = {d.batch, d.block_len, d.nheads, BDLM_HEADDIM};
    const at::Tensor yn = out(a[17], shape, t.x), yc = opt_out(a[16], shape, t.x);
    float *ynp = ptr<float>(yn), *ycp = opt_ptr(yc);
    const void *x = ptr(t.x), *dt = ptr(t.dt), *B = ptr(t.B), *C = ptr(t.C);
    const void *x2 = ptr(r.x), *dt2 = ptr(r.dt), *B2 = ptr(r.B), *C2 = ptr(r.C);
    return enqueue(pair(yn, yc), [&] {
        return bdlm_commit_step(&d, x, dt, A, B, C, D, Dr, x2, dt2, B2, C2, h, ns, sl.p, nc.p, nb.p, want, ycp, ynp, s);
    });
} BDLM_END

// The convolution's weights, biases and cached rows.
struct Conv {
    const float *w, *b;
    float *rows;
    Conv(PyObject *pw, PyObject *pb, PyObject *prows, const bdlm_desc_t &d, int64_t nslots) {
        const int64_t ch = d.nheads * BDLM_HEADDIM + 2 * d.ngroups * d.dstate;
        const at::Tensor &tw = tensor(pw), &tr = tensor(prows);
        need(tw.scalar_type() == at::kFloat && tw.dim() == 2 && tw.size(0) == ch && tw.size(1) == 4 && tw.is_contiguous());
        need(tr.scalar_type() == at::kFloat && tr.dim() == 3 && tr.size(0) == nslots && tr.size(1) == 3 &&
             tr.size(2) == ch && tr.is_contiguous());
        w = ptr<float>(tw);
        b = vec(pb, ch);
        rows = ptr<float>(tr);
    }
};

// x dt A B C D D_rev conv_w conv_b conv_pool h_pool y slot_idx stream workspace
BDLM_ENTRY(conv_block_step, 15) {
    Acts t(a[0], a[1], a[3], a[4]);
    const bdlm_desc_t &d = t.d;
    const float *A = vec(a[2], d.nheads), *D = vec(a[5], d.nheads), *Dr = vec(a[6], d.nheads);
    int64_t ns, bytes = 0;
    const float *h = pool(a[10], d, &ns);
    const Conv c(a[7], a[8], a[9], d, ns);
    const Slots sl(a[12], d.batch);
    void *s = stream_of(a[13]);
    need(bdlm_conv_workspace(&d, &bytes) == BDLM_OK);
    const at::Tensor y = out(a[11], {d.batch, d.block_len, d.nheads, BDLM_HEADDIM}, t.x);
    const Workspace ws(a[14], bytes, t.x);
    float *yp = ptr<float>(y);
    const void *x = ptr(t.x), *dt = ptr(t.dt), *B = ptr(t.B), *C = ptr(t.C);
    return enqueue(item(y), [&] {
        return bdlm_conv_block_step(&d, x, dt, A, B, C, D, Dr, c.w, c.b, c.rows, h, ns, sl.p, yp, ws.p, ws.bytes, s);
    });
} BDLM_END

// x dt A B C D D_rev conv_w conv_b conv_pool h_pool n_committed n_blocks expected slot_idx y_clean stream workspace
BDLM_ENTRY(conv_commit_boundary, 18) {
    Acts t(a[0], a[1], a[3], a[4]);
    const bdlm_desc_t &d = t.d;
    const float *A = vec(a[2], d.nheads), *D = vec(a[5], d.nheads), *Dr = vec(a[6], d.nheads);
    int64_t ns, bytes = 0;
    float *h = pool(a[10], d, &ns);
    const Conv c(a[7], a[8], a[9], d, ns);
    Books nc(a[11], ns), nb(a[12], ns);
    const int64_t want = integer(a[13]);
    const Slots sl(a[14], d.batch);
    void *s = stream_of(a[16]);
    need(bdlm_conv_workspace(&d, &bytes) == BDLM_OK);
    const at::Tensor y = opt_out(a[15], {d.batch, d.block_len, d.nheads, BDLM_HEADDIM}, t.x);
    const Workspace ws(a[17], bytes, t.x);
    float *yp = opt_ptr(y);
    const void *x = ptr(t.x), *dt = ptr(t.dt), *B = ptr(t.B), *C = ptr(t.C);
    return enqueue(item(y), [&] {
        return bdlm_conv_commit_boundary(&d, x, dt, A, B, C, D, Dr, c.w, c.b, c.rows, h, ns, sl.p, nc.p, nb.p, want, yp,
                                         ws.p, ws.bytes, s);
    });
} BDLM_END

// x dt A B C D D_rev y stream workspace
BDLM_ENTRY(scan_full_window, 10) {
    Acts t(a[0], a[1], a[3], a[4]);
    const bdlm_desc_t &d = t.d;
    const float *A = vec(a[2], d.nheads), *D = vec(a[5], d.nheads), *Dr = vec(a[6], d.nheads);
    int64_t bytes = 0;
    void *s = stream_of(a[8]);
    need(bdlm_full_window_workspace(&d, &bytes) == BDLM_OK);
    const at::Tensor y = out(a[7], {d.batch, d.block_len, d.nheads, BDLM_HEADDIM}, t.x);
    const Workspace ws(a[9], bytes, t.x);
    float *yp = ptr<float>(y);
    const void *x = ptr(t.x), *dt = ptr(t.dt), *B = ptr(t.B), *C = ptr(t.C);
    return enqueue(item(y), [&] { return bdlm_scan_full_window(&d, x, dt, A, B, C, D, Dr, yp, ws.p, ws.bytes, s); });
} BDLM_END

// x dt A B C D h_pool n_committed n_blocks expected blocks_in_prefix slot_idx y_fwd stream workspace
BDLM_ENTRY(prefill, 15) {
    Acts t(a[0], a[1], a[3], a[4]);
    const bdlm_desc_t &d = t.d;
    const float *A = vec(a[2], d.nheads), *D = vec(a[5], d.nheads);
    int64_t ns, bytes = 0;
    float *h = pool(a[6], d, &ns);
    Books nc(a[7], ns), nb(a[8], ns);
    const int64_t want = integer(a[9]), blocks = integer(a[10]);
    const Slots sl(a[11], d.batch);
    void *s = stream_of(a[13]);
    need(bdlm_prefill_workspace(&d, &bytes) == BDLM_OK);
    const at::Tensor y = opt_out(a[12], {d.batch, d.block_len, d.nheads, BDLM_HEADDIM}, t.x);
    const Workspace ws(a[14], bytes, t.x);
    float *yp = opt_ptr(y);
    const void *x = ptr(t.x), *dt = ptr(t.dt), *B = ptr(t.B), *C = ptr(t.C);
    return enqueue(item(y), [&] {
        return bdlm_prefill(&d, x, dt, A, B, C, D, h, ns, sl.p, nc.p, nb.p, want, blocks, yp, ws.p, ws.bytes, s);
    });
} BDLM_END

// x dt A B C D h_pool n_committed n_blocks expected blocks_in_prefix slot_idx y_fwd stream
BDLM_ENTRY(prefill_noalloc, 14) {
    Acts t(a[0], a[1], a[3], a[4]);
    const bdlm_desc_t &d = t.d;
    const float *A = vec(a[2], d.nheads), *D = vec(a[5], d.nheads);
    int64_t ns;
    float *h = pool(a[6], d, &ns);
    Books nc(a[7], ns), nb(a[8], ns);
    const int64_t want = integer(a[9]), blocks = integer(a[10]);
    const Slots sl(a[11], d.batch);
    void *s = stream_of(a[13]);
    need(a[12] != Py_True);
    const at::Tensor y = opt_out(a[12], {d.batch, d.block_len, d.nheads, BDLM_HEADDIM}, t.x);
    float *yp = opt_ptr(y);
    const void *x = ptr(t.x), *dt = ptr(t.dt), *B = ptr(t.B), *C = ptr(t.C);
    return enqueue(item(y), [&] {
        return bdlm_prefill_noalloc(&d, x, dt, A, B, C, D, h, ns, sl.p, nc.p, nb.p, want, blocks, yp, s);
    });
} BDLM_END

// y z norm_w eps ngroups out stream
BDLM_ENTRY(gated_rmsnorm, 7) {
    const at::Tensor &y = tensor(a[0]), &z = tensor(a[1]);
    need(y.scalar_type() == at::kFloat && y.is_contiguous() && (y.dim() == 3 || y.dim() == 4));
    const int64_t b = y.size(0), L = y.size(1), nch = y.dim() == 4 ? y.size(2) * y.size(3) : y.size(2);
    need(b * L > 0 && nch > 0 && nch % BDLM_HEADDIM == 0);
    need(z.dim() == 3 && z.size(0) == b && z.size(1) == L && z.size(2) == nch && z.stride(2) == 1);
    need(z.scalar_type() == at::kBFloat16 || z.scalar_type() == at::kFloat);
    const float *w = vec(a[2], nch);
    need(PyFloat_CheckExact(a[3]));
    const float eps = static_cast<float>(PyFloat_AS_DOUBLE(a[3]));
    const int64_t groups = integer(a[4]);
    void *s = stream_of(a[6]);
    at::Tensor o;
    if (a[5] == Py_None) {
        const Unlocked u;
        o = at::empty_like(y);
    } else {
        need(a[5] != Py_True);
        o = out(a[5], y.sizes(), y);
    }
    const float *yp = ptr<float>(y);
    const void *zp = ptr(z);
    float *op = ptr<float>(o);
    const int64_t zb = z.stride(0), zt = z.stride(1);
    const int32_t zd = z.scalar_type() == at::kBFloat16 ? BDLM_DTYPE_BF16 : BDLM_DTYPE_F32;
    return enqueue(item(o), [&] {
        return bdlm_gated_rmsnorm(b, L, nch / BDLM_HEADDIM, groups, zd, yp, zp, zb, zt, w, eps, op, s);
    });
} BDLM_END

#define BDLM_METHOD(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    BDLM_METHOD(scan_block_step), BDLM_METHOD(scan_block_step_sep), BDLM_METHOD(commit_boundary),
    BDLM_METHOD(commit_step), BDLM_METHOD(conv_block_step), BDLM_METHOD(conv_commit_boundary),
    BDLM_METHOD(scan_full_window), BDLM_METHOD(prefill),
    BDLM_METHOD(prefill_noalloc), BDLM_METHOD(gated_rmsnorm), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_bind", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__bind() {
    PyObject *np = PyImport_ImportModule("numpy");
    if (!np) return nullptr;
    g_ndarray = PyObject_GetAttrString(np, "ndarray");
    Py_DECREF(np);
    return g_ndarray ? PyModule_Create(&module) : nullptr;
}
