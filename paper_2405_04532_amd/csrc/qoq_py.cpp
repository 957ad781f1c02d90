// Native argument marshalling of the calls that a serving loop makes per layer: checks the tensors, allocates the results,
// takes the current stream and calls the C ABI.  The same checks and results as their Python counterparts in api.py had;
// through ctypes a call of the activation quantizer took 10.6 us of host time and a GEMM 7.7 us, more than their kernels at
// decode sizes, of which the launch itself is about 2 us (the rest: argument objects, torch.empty, the stream lookup).
// Nothing is kept between calls.  The interpreter lock is released around the library call, as ctypes does.
#include <Python.h>

#include <algorithm>

#include <ATen/ops/empty.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/qoq_w4a8.h"
#include "qoq_workspace.h"

namespace {

PyObject* g_raise_status = nullptr;             // Python callable that raises the error of a status code

bool counted(Py_ssize_t got, Py_ssize_t want)
{
    if (got == want) return true;
    PyErr_Format(PyExc_TypeError, "expected %zd arguments, got %zd", want, got);
    return false;
}

// a tensor argument; nullptr with an exception set if it is something else
const at::Tensor* tensor(PyObject* o, const char* name)
{
    if (THPVariable_Check(o)) return &THPVariable_Unpack(o);
    PyErr_Format(PyExc_TypeError, "%s: expected a tensor", name);
    return nullptr;
}

// a contiguous tensor of this type on the GPU
const at::Tensor* dev_tensor(PyObject* o, at::ScalarType dtype, const char* name)
{
    const at::Tensor* t = tensor(o, name);
    if (!t || (t->is_cuda() && t->scalar_type() == dtype && t->is_contiguous())) return t;
    const char* type = dtype == at::kHalf ? "torch.float16" : dtype == at::kChar ? "torch.int8" : dtype == at::kInt ? "torch.int32" : "torch.float32";
    PyErr_Format(PyExc_TypeError, "%s: expected a contiguous %s tensor on the GPU", name, type);
    return nullptr;
}

bool has_dims(const at::Tensor& t, int64_t dims, const char* name)
{
    if (t.dim() == dims) return true;
    PyErr_Format(PyExc_ValueError, "%s: expected %lld dimensions, got %lld", name, (long long)dims, (long long)t.dim());
    return false;
}

// address of a tensor or None; false with an exception set for anything else
bool pointer(PyObject* o, const char* name, void** p)
{
    *p = nullptr;
    if (o == Py_None) return true;
    const at::Tensor* t = tensor(o, name);
    if (!t) return false;
    *p = t->data_ptr();
    return true;
}

bool integer(PyObject* o, int64_t* v)
{
    *v = PyLong_AsLongLong(o);
    return !(*v == -1 && PyErr_Occurred());
}

// a truth value, as `if o:` takes it; false with the exception set if it has none
bool flag(PyObject* o, bool* v)
{
    const int t = PyObject_IsTrue(o);
    *v = t == 1;
    return t >= 0;
}

bool number(PyObject* o, double* v)             // as float(o) takes it
{
    PyObject* f = PyNumber_Float(o);
    if (!f) return false;
    *v = PyFloat_AS_DOUBLE(f);
    Py_DECREF(f);
    return true;
}

void* stream_of(const at::Tensor& t) { return c10::hip::getCurrentHIPStream(t.get_device()).stream(); }

at::Tensor new_like(const at::Tensor& on, at::IntArrayRef shape, at::ScalarType dtype)
{
    return at::empty(shape, at::TensorOptions().dtype(dtype).device(on.device()));
}

template <class F>
bool call(F&& f)                                // true: QOQ_OK; false: the status's exception is set
{
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = f();
    Py_END_ALLOW_THREADS
    if (status == QOQ_OK) return true;
    PyObject* r = PyObject_CallFunction(g_raise_status, "i", status);
    Py_XDECREF(r);
    return false;
}

// the results of a quantizing call, in the order in which api.py returns them
struct Quantized {
    at::Tensor y, qx, sx, rowsum, tx;
    Quantized(const at::Tensor& on, int64_t M, int64_t K, bool want_y, bool want_rowsum, bool want_tx)
    {
        if (want_y) y = new_like(on, {M, K}, at::kHalf);
        qx = new_like(on, {M, K}, at::kChar);
        sx = new_like(on, {M}, at::kHalf);
        if (want_rowsum) rowsum = new_like(on, {M}, at::kInt);
        if (want_tx) tx = new_like(on, {M}, at::kFloat);
    }
    static void* at_or_null(const at::Tensor& t) { return t.defined() ? t.data_ptr() : nullptr; }
    static PyObject* wrap(const at::Tensor& t)
    {
        if (t.defined()) return THPVariable_Wrap(t);
        Py_RETURN_NONE;
    }
    void* y_ptr() const { return at_or_null(y); }
    int8_t* qx_ptr() const { return static_cast<int8_t*>(qx.data_ptr()); }
    void* sx_ptr() const { return sx.data_ptr(); }
    int32_t* rowsum_ptr() const { return static_cast<int32_t*>(at_or_null(rowsum)); }
    float* tx_ptr() const { return static_cast<float*>(at_or_null(tx)); }
    PyObject* result(bool with_y) const
    {
        return with_y ? Py_BuildValue("NNNNN", wrap(y), wrap(qx), wrap(sx), wrap(rowsum), wrap(tx))
                      : Py_BuildValue("NNNN", wrap(qx), wrap(sx), wrap(rowsum), wrap(tx));
    }
};

PyObject* quant_act(PyObject*, PyObject* const* a, Py_ssize_t n)    // x, want_rowsum, want_tx
{
    HANDLE_TH_ERRORS
    if (!counted(n, 3)) return nullptr;
    const at::Tensor* x = dev_tensor(a[0], at::kHalf, "x");
    bool want_rowsum, want_tx;
    if (!x || !has_dims(*x, 2, "x") || !flag(a[1], &want_rowsum) || !flag(a[2], &want_tx)) return nullptr;
    const int64_t M = x->size(0), K = x->size(1);
    const Quantized q(*x, M, K, false, want_rowsum, want_tx);
    void* s = stream_of(*x);
    const void* xp = x->data_ptr();
    if (!call([&] { return qoq_quant_act_per_token(xp, M, K, q.qx_ptr(), q.sx_ptr(), q.rowsum_ptr(), q.tx_ptr(), s); })) return nullptr;
    return q.result(false);
    END_HANDLE_TH_ERRORS
}

PyObject* quant_act_reordered(PyObject*, PyObject* const* a, Py_ssize_t n)    // x, perm, want_rowsum, want_tx
{
    HANDLE_TH_ERRORS
    if (!counted(n, 4)) return nullptr;
    const at::Tensor* x = dev_tensor(a[0], at::kHalf, "x");
    if (!x) return nullptr;
    const at::Tensor* perm = dev_tensor(a[1], at::kInt, "perm");
    bool want_rowsum, want_tx;
    if (!perm || !has_dims(*x, 2, "x") || !flag(a[2], &want_rowsum) || !flag(a[3], &want_tx)) return nullptr;
    const int64_t M = x->size(0), K = x->size(1);
    const Quantized q(*x, M, K, false, want_rowsum, want_tx);
    void* s = stream_of(*x);
    const void* xp = x->data_ptr();
    const int32_t* pp = static_cast<const int32_t*>(perm->data_ptr());
    if (!call([&] { return qoq_quant_act_per_token_reordered(xp, pp, M, K, q.qx_ptr(), q.sx_ptr(), q.rowsum_ptr(), q.tx_ptr(), s); }))
        return nullptr;
    return q.result(false);
    END_HANDLE_TH_ERRORS
}

PyObject* rmsnorm_quant(PyObject*, PyObject* const* a, Py_ssize_t n)    // x, gamma, eps, want_y, want_rowsum, want_tx
{
    HANDLE_TH_ERRORS
    if (!counted(n, 6)) return nullptr;
    const at::Tensor* x = dev_tensor(a[0], at::kHalf, "x");
    if (!x) return nullptr;
    const at::Tensor* gamma = dev_tensor(a[1], at::kHalf, "gamma");
    bool want_y, want_rowsum, want_tx;
    double eps;
    if (!gamma || !has_dims(*x, 2, "x") || !number(a[2], &eps) || !flag(a[3], &want_y) || !flag(a[4], &want_rowsum) || !flag(a[5], &want_tx))
        return nullptr;
    const int64_t M = x->size(0), K = x->size(1);
    const Quantized q(*x, M, K, want_y, want_rowsum, want_tx);
    void* s = stream_of(*x);
    const void *xp = x->data_ptr(), *gp = gamma->data_ptr();
    if (!call([&] { return qoq_rmsnorm_quant(xp, gp, eps, M, K, q.y_ptr(), q.qx_ptr(), q.sx_ptr(), q.rowsum_ptr(), q.tx_ptr(), s); }))
        return nullptr;
    return q.result(true);
    END_HANDLE_TH_ERRORS
}

PyObject* silu_mul_quant(PyObject*, PyObject* const* a, Py_ssize_t n)    // gate_up, want_y, want_rowsum, want_tx
{
    HANDLE_TH_ERRORS
    if (!counted(n, 4)) return nullptr;
    const at::Tensor* x = dev_tensor(a[0], at::kHalf, "gate_up");
    bool want_y, want_rowsum, want_tx;
    if (!x || !has_dims(*x, 2, "gate_up") || !flag(a[1], &want_y) || !flag(a[2], &want_rowsum) || !flag(a[3], &want_tx)) return nullptr;
    const int64_t M = x->size(0), K = x->size(1) / 2;
    const Quantized q(*x, M, K, want_y, want_rowsum, want_tx);
    void* s = stream_of(*x);
    const void* xp = x->data_ptr();
    if (!call([&] { return qoq_silu_mul_quant(xp, M, K, q.y_ptr(), q.qx_ptr(), q.sx_ptr(), q.rowsum_ptr(), q.tx_ptr(), s); })) return nullptr;
    return q.result(true);
    END_HANDLE_TH_ERRORS
}

// the caller's tensor, or a new one of this shape; `owned` keeps the new one alive and becomes the result
PyObject* given_or_new(PyObject* given, const at::Tensor& on, at::IntArrayRef shape, at::ScalarType dtype, const char* name, void** p)
{
    if (given == Py_None) {
        at::Tensor t = new_like(on, shape, dtype);
        *p = t.data_ptr();
        return THPVariable_Wrap(std::move(t));
    }
    if (!pointer(given, name, p)) return nullptr;
    Py_INCREF(given);
    return given;
}

struct Ref {                                    // an owned reference that is dropped unless it is released
    PyObject* o;
    explicit Ref(PyObject* p) : o(p) {}
    ~Ref() { Py_XDECREF(o); }
    PyObject* release() { PyObject* r = o; o = nullptr; return r; }
    explicit operator bool() const { return o != nullptr; }
};

// Workspace of a GEMM call: the caller's, or one of what the call exchanges, its counters zeroed on the stream (zeroing all of it, as
// a workspace that is kept is prepared, took 4 to 11 us more for 12 to 39 MB).
struct Workspace {
    at::Tensor own;
    void* ptr = nullptr;
    size_t bytes = 0;
    bool ready(PyObject* given, const at::Tensor& on, int64_t M, int64_t N, int64_t K, int64_t mode, void* stream)
    {
        if (given != Py_None) {
            const at::Tensor* t = tensor(given, "workspace");
            if (!t) return false;
            ptr = t->data_ptr();
            bytes = (size_t)t->numel() * t->element_size();
            return true;
        }
        bytes = qoq::gemm_fresh_workspace_bytes(M, N, K, (int)mode);
        if (!bytes) return true;
        own = new_like(on, {(int64_t)bytes}, at::kByte);
        ptr = own.data_ptr();
        return call([&] { return qoq_gemm_workspace_prepare(ptr, std::min(bytes, (size_t)QOQ_GEMM_COUNTER_BYTES), stream); });
    }
};

PyObject* w4a8_gemm(PyObject*, PyObject* const* a, Py_ssize_t n)    // qx, sx, packed, N, mode, rowsum, out, workspace
{
    HANDLE_TH_ERRORS
    if (!counted(n, 8)) return nullptr;
    const at::Tensor* qx = dev_tensor(a[0], at::kChar, "qx");
    int64_t N, mode;
    void *sx, *packed, *rowsum, *out;
    if (!qx || !has_dims(*qx, 2, "qx") || !integer(a[3], &N) || !integer(a[4], &mode) || !pointer(a[1], "sx", &sx) ||
        !pointer(a[2], "packed", &packed) || !pointer(a[5], "rowsum", &rowsum))
        return nullptr;
    const int64_t M = qx->size(0), K = qx->size(1);
    void* s = stream_of(*qx);
    Ref res(given_or_new(a[6], *qx, {M, N}, at::kHalf, "out", &out));
    Workspace ws;
    if (!res || !ws.ready(a[7], *qx, M, N, K, mode, s)) return nullptr;
    const int8_t* xp = static_cast<const int8_t*>(qx->data_ptr());
    if (!call([&] { return qoq_w4a8_gemm(xp, sx, static_cast<int32_t*>(rowsum), packed, M, N, K, (int)mode, out, ws.ptr, ws.bytes, s); }))
        return nullptr;
    return res.release();
    END_HANDLE_TH_ERRORS
}

PyObject* w4a8_gemm_noalloc(PyObject*, PyObject* const* a, Py_ssize_t n)    // qx, sx, packed, N, out, mode, rowsum
{
    HANDLE_TH_ERRORS
    if (!counted(n, 7)) return nullptr;
    const at::Tensor* qx = dev_tensor(a[0], at::kChar, "qx");
    if (!qx) return nullptr;
    const at::Tensor* out = dev_tensor(a[4], at::kHalf, "out");
    int64_t N, mode;
    void *sx, *packed, *rowsum;
    if (!out || !has_dims(*qx, 2, "qx") || !integer(a[3], &N) || !integer(a[5], &mode) || !pointer(a[1], "sx", &sx) ||
        !pointer(a[2], "packed", &packed) || !pointer(a[6], "rowsum", &rowsum))
        return nullptr;
    const int64_t M = qx->size(0), K = qx->size(1);
    void *s = stream_of(*qx), *op = out->data_ptr();
    const int8_t* xp = static_cast<const int8_t*>(qx->data_ptr());
    if (!call([&] { return qoq_w4a8_gemm_noalloc(xp, sx, static_cast<int32_t*>(rowsum), packed, M, N, K, (int)mode, op, s); })) return nullptr;
    Py_INCREF(a[4]);
    return a[4];
    END_HANDLE_TH_ERRORS
}

PyObject* w4a8_gemm_token_sum(PyObject*, PyObject* const* a, Py_ssize_t n)    // qx, sx, tx, packed, N, out, workspace
{
    HANDLE_TH_ERRORS
    if (!counted(n, 7)) return nullptr;
    const at::Tensor* qx = dev_tensor(a[0], at::kChar, "qx");
    if (!qx) return nullptr;
    const at::Tensor* tx = dev_tensor(a[2], at::kFloat, "tx");
    int64_t N;
    void *sx, *packed, *out;
    if (!tx || !has_dims(*qx, 2, "qx") || !integer(a[4], &N) || !pointer(a[1], "sx", &sx) || !pointer(a[3], "packed", &packed)) return nullptr;
    const int64_t M = qx->size(0), K = qx->size(1);
    void* s = stream_of(*qx);
    Ref res(given_or_new(a[5], *qx, {M, N}, at::kHalf, "out", &out));
    Workspace ws;
    if (!res || !ws.ready(a[6], *qx, M, N, K, QOQ_PER_CHANNEL, s)) return nullptr;
    const int8_t* xp = static_cast<const int8_t*>(qx->data_ptr());
    const float* tp = static_cast<const float*>(tx->data_ptr());
    if (!call([&] { return qoq_w4a8_gemm_token_sum(xp, sx, tp, packed, M, N, K, out, ws.ptr, ws.bytes, s); })) return nullptr;
    return res.release();
    END_HANDLE_TH_ERRORS
}

PyObject* w4a8_linear(PyObject*, PyObject* const* a, Py_ssize_t n)    // x, packed, N, mode, out, qx, sx, rowsum, workspace
{
    HANDLE_TH_ERRORS
    if (!counted(n, 9)) return nullptr;
    const at::Tensor* x = dev_tensor(a[0], at::kHalf, "x");
    int64_t N, mode;
    void *packed, *out, *qx, *sx, *rowsum;
    if (!x || !has_dims(*x, 2, "x") || !integer(a[2], &N) || !integer(a[3], &mode) || !pointer(a[1], "packed", &packed)) return nullptr;
    const int64_t M = x->size(0), K = x->size(1);
    void* s = stream_of(*x);
    Ref r_out(given_or_new(a[4], *x, {M, N}, at::kHalf, "out", &out));
    Ref r_qx(r_out ? given_or_new(a[5], *x, {M, K}, at::kChar, "qx", &qx) : nullptr);
    Ref r_sx(r_qx ? given_or_new(a[6], *x, {M}, at::kHalf, "sx", &sx) : nullptr);
    Ref r_rs(r_sx ? given_or_new(a[7], *x, {M}, at::kInt, "rowsum", &rowsum) : nullptr);
    Workspace ws;
    if (!r_rs || !ws.ready(a[8], *x, M, N, K, mode, s)) return nullptr;
    const void* xp = x->data_ptr();
    if (!call([&] {
            return qoq_w4a8_linear(xp, packed, M, N, K, (int)mode, out, static_cast<int8_t*>(qx), sx, static_cast<int32_t*>(rowsum), ws.ptr,
                                   ws.bytes, s);
        }))
        return nullptr;
    return Py_BuildValue("NNNN", r_out.release(), r_qx.release(), r_sx.release(), r_rs.release());
    END_HANDLE_TH_ERRORS
}

PyObject* kv4_append(PyObject*, PyObject* const* a, Py_ssize_t n)    // cache, k, v, positions, S_max
{
    HANDLE_TH_ERRORS
    if (!counted(n, 5)) return nullptr;
    const at::Tensor* k = dev_tensor(a[1], at::kHalf, "k");
    const at::Tensor* v = k ? dev_tensor(a[2], at::kHalf, "v") : nullptr;
    const at::Tensor* pos = v ? dev_tensor(a[3], at::kInt, "positions") : nullptr;
    int64_t S_max;
    void* cache;
    if (!pos || !has_dims(*k, 4, "k") || !integer(a[4], &S_max) || !pointer(a[0], "cache", &cache)) return nullptr;
    const int64_t B = k->size(0), T = k->size(1), Hkv = k->size(2), D = k->size(3);
    void* s = stream_of(*k);
    const void *kp = k->data_ptr(), *vp = v->data_ptr();
    const int32_t* pp = static_cast<const int32_t*>(pos->data_ptr());
    if (!call([&] { return qoq_kv4_append(kp, vp, pp, B, T, Hkv, D, S_max, cache, s); })) return nullptr;
    Py_RETURN_NONE;
    END_HANDLE_TH_ERRORS
}

PyObject* kv4_attention_decode(PyObject*, PyObject* const* a, Py_ssize_t n)    // q, cache, seq_lens, Hkv, S_max, out, workspace
{
    HANDLE_TH_ERRORS
    if (!counted(n, 7)) return nullptr;
    const at::Tensor* q = dev_tensor(a[0], at::kHalf, "q");
    const at::Tensor* lens = q ? dev_tensor(a[2], at::kInt, "seq_lens") : nullptr;
    int64_t Hkv, S_max;
    void *cache, *out;
    if (!lens || !has_dims(*q, 3, "q") || !integer(a[3], &Hkv) || !integer(a[4], &S_max) || !pointer(a[1], "cache", &cache)) return nullptr;
    const int64_t B = q->size(0), H = q->size(1), D = q->size(2);
    void* s = stream_of(*q);
    Ref res(given_or_new(a[5], *q, {B, H, D}, at::kHalf, "out", &out));
    if (!res) return nullptr;
    const void* qp = q->data_ptr();
    const int32_t* lp = static_cast<const int32_t*>(lens->data_ptr());
    if (a[6] == Py_None) {
        if (!call([&] { return qoq_kv4_attention_decode(qp, cache, lp, B, H, Hkv, D, S_max, out, s); })) return nullptr;
    } else {
        const at::Tensor* ws = tensor(a[6], "workspace");
        if (!ws) return nullptr;
        void* wp = ws->data_ptr();
        const size_t bytes = (size_t)ws->numel();
        if (!call([&] { return qoq_kv4_attention_decode_split(qp, cache, lp, B, H, Hkv, D, S_max, out, wp, bytes, s); })) return nullptr;
    }
    return res.release();
    END_HANDLE_TH_ERRORS
}

PyObject* set_raise_status(PyObject*, PyObject* f)
{
    Py_INCREF(f);
    Py_XSETREF(g_raise_status, f);
    Py_RETURN_NONE;
}

// The order of salient channels, and whether it is one: the kernel says so in pinned host memory.  The call returns when the order is complete,
// which callers may then use, and salience reuse, on any stream.  (Returning with the verdict, which is there when the others begin to
// sort, 4096 x 14336 reordered and packed takes 96 us a pass and not 109, but other streams then read an order that is not there yet.  Flags that
// the sorting workgroups set when their parts are in memory, polled in place of the stream, 108; with a system-wide fence each 113.)
PyObject* channel_order(PyObject*, PyObject* const* a, Py_ssize_t n)    // salience
{
    HANDLE_TH_ERRORS
    if (!counted(n, 1)) return nullptr;
    const at::Tensor* sal = dev_tensor(a[0], at::kFloat, "salience");
    if (!sal) return nullptr;
    const hipStream_t s = static_cast<hipStream_t>(stream_of(*sal));
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &capture) != hipSuccess || capture != hipStreamCaptureStatusNone) {
        (void)hipGetLastError();                // (the default stream beside a capture: not the next launch's error)
        PyErr_SetString(PyExc_RuntimeError, "channel_order reads a result on the host: not while the stream is being captured");
        return nullptr;
    }
    const int64_t K = sal->numel();
    at::Tensor perm = new_like(*sal, {K}, at::kInt);
    at::Tensor pinned = at::empty({1}, at::TensorOptions().dtype(at::kInt).pinned_memory(true));
    int32_t* verdict = static_cast<int32_t*>(pinned.data_ptr());
    const float* sp = static_cast<const float*>(sal->data_ptr());
    int32_t* pp = static_cast<int32_t*>(perm.data_ptr());
    __atomic_store_n(verdict, -1, __ATOMIC_RELEASE);
    if (!call([&] {
            const int status = qoq_channel_order(sp, K, pp, verdict, s);
            if (status != QOQ_OK) return status;
            if (hipStreamSynchronize(s) != hipSuccess) return (int)QOQ_ERR_HIP;
            const int v = __atomic_load_n(verdict, __ATOMIC_ACQUIRE);
            return v == 0 ? (int)QOQ_OK : v > 0 ? (int)QOQ_ERR_SHAPE : (int)QOQ_ERR_HIP;
        }))
        return nullptr;
    return THPVariable_Wrap(perm);
    END_HANDLE_TH_ERRORS
}

#define FAST(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {FAST(quant_act), FAST(quant_act_reordered), FAST(rmsnorm_quant), FAST(silu_mul_quant), FAST(w4a8_gemm),
                         FAST(w4a8_gemm_noalloc), FAST(w4a8_gemm_token_sum), FAST(w4a8_linear), FAST(kv4_append), FAST(kv4_attention_decode), FAST(channel_order),
                         {"set_raise_status", set_raise_status, METH_O, nullptr}, {nullptr, nullptr, 0, nullptr}};
#undef FAST
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_qoq_py", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// torch_version: the torch whose classes this was compiled against; api.py refuses any other.
PyMODINIT_FUNC PyInit__qoq_py(void)
{
    PyObject* m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "torch_version", QOQ_TORCH_VERSION) != 0) Py_CLEAR(m);
    return m;
}
