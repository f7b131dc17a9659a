// Native marshalling of the binding's calls: torch tensors -> (pointer, strides) descriptors -> one call of the C library.
//
// What bounds a small call is the host: reading the properties of its tensors through Python objects and building ctypes
// structures took 5 ... 15 us of a call that launches one or two kernels of 3 ... 10 us.  Here a tensor costs a few loads.
// Every function takes the arguments of the Python function of the same name, positionally, and returns the status of the
// library's call, or None where an argument is not of the plain form handled here (exact torch tensors in device memory with the
// expected type, lists, tuples and numbers).  Nothing has been enqueued then, and the caller takes its general path, which says
// what is wrong or converts it.  So errors have one place, and a tensor that is more than memory with strides (a subclass, a
// batched or functional wrapper) never gets past its own dispatch here.
// us on the host per step, ctypes -> here: 4 x 512 tokens, 8 anchors, weights 30.2 -> 7.8; two segments' weights and update 41.9 -> 16.8; 77
// tokens, 6 anchors, both calls 32.5 -> 18.4; one decoded token, two launches 12.5 -> 9.9; a whole step of 2 layers (three
// calls) 35.2 -> 19.9, which took the step from 30.4 to 20.2 us.
#include <torch/csrc/Dtype.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cxxabi.h>

#include <algorithm>
#include <climits>

#include "kvcomm.h"

namespace {

struct Decline {};   // not of the plain form: the caller's general path takes over

constexpr int kMaxAnchors = KVCOMM_MAX_ANCHORS, kMaxBatch = KVCOMM_MAX_BATCH;

// The library's entry points and what is needed of Python, set once by bind().
struct Library {
    decltype(&kvcomm_weight_slots) weight_slots;
    decltype(&kvcomm_suffix_attn_workspace) attn_workspace;
    decltype(&kvcomm_anchor_weights_rule) anchor_weights_rule;
    decltype(&kvcomm_anchor_weights_batch) anchor_weights_batch;
    decltype(&kvcomm_align_kv_batch) align_kv_batch;
    decltype(&kvcomm_align_kv_batch_beside) align_kv_batch_beside;
    decltype(&kvcomm_align_kv_q8_batch) align_kv_q8_batch;
    decltype(&kvcomm_align_kv) align_kv;
    decltype(&kvcomm_align_kv_q8) align_kv_q8;
    decltype(&kvcomm_suffix_attn) suffix_attn;
    decltype(&kvcomm_suffix_attn_confined_ws) suffix_attn_confined_ws;
    decltype(&kvcomm_anchor_predict) anchor_predict;
    decltype(&kvcomm_capture_offsets) capture_offsets;
    decltype(&kvcomm_quantize_deltas) quantize_deltas;
    PyObject *model_type, *current_device, *current_stream;
} lib;

struct Names {
    PyObject *n_layers, *n_kv_heads, *n_q_heads, *head_dim, *dtype, *rope_theta, *cuda_stream;
    PyObject *seg_base_k, *anchor_base_k, *anchor_len, *base_k, *base_v, *anchor_dk, *anchor_dv, *anchor_dk8, *anchor_dv8, *scale_k,
        *scale_v, *weights, *delta_pos, *anchor_delta_pos, *out_k, *out_v;
} names;

// ------------------------------------------------------------------------------------------ plain values
int32_t as_int(PyObject *o)
{
    if (!PyLong_CheckExact(o)) throw Decline{};
    int overflow = 0;
    const long v = PyLong_AsLongAndOverflow(o, &overflow);
    if (overflow || v < INT32_MIN || v > INT32_MAX) throw Decline{};
    return (int32_t)v;
}

double as_double(PyObject *o)
{
    if (PyFloat_CheckExact(o)) return PyFloat_AS_DOUBLE(o);
    return (double)as_int(o);
}

// A plain strided tensor in device memory.  Functional and batched wrappers, tensors with symbolic sizes and subclasses have
// more to say about their data than a pointer.
const at::Tensor &as_tensor(PyObject *o)
{
    if (!THPVariable_CheckExact(o)) throw Decline{};
    const at::Tensor &t = THPVariable_Unpack(o);
    constexpr c10::DispatchKeySet wrapped({c10::DispatchKey::Python, c10::DispatchKey::PythonTLSSnapshot, c10::DispatchKey::FuncTorchBatched,
                                           c10::DispatchKey::FuncTorchGradWrapper, c10::DispatchKey::Functionalize,
                                           c10::DispatchKey::ZeroTensor});
    if (!t.defined() || !t.is_cuda() || t.layout() != at::kStrided || t.key_set().has_any(wrapped) ||
        t.unsafeGetTensorImpl()->has_symbolic_sizes_strides() || !t.has_storage())
        throw Decline{};
    return t;
}

struct Call {   // the model of a call and its tensors' type
    kvcomm_model m;
    at::ScalarType dtype;
    explicit Call(PyObject *model)
    {
        if (Py_TYPE(model) != (PyTypeObject *)lib.model_type) throw Decline{};
        auto get = [&](PyObject *name) {
            PyObject *v = PyObject_GetAttr(model, name);
            if (!v) throw Decline{};
            return py(v);
        };
        m.n_layers = as_int(get(names.n_layers).o);
        m.n_kv_heads = as_int(get(names.n_kv_heads).o);
        m.n_q_heads = as_int(get(names.n_q_heads).o);
        m.head_dim = as_int(get(names.head_dim).o);
        m.rope_theta = as_double(get(names.rope_theta).o);
        const py d = get(names.dtype);
        if (!THPDtype_Check(d.o)) throw Decline{};
        dtype = reinterpret_cast<THPDtype *>(d.o)->scalar_type;
        if (dtype != at::kBFloat16 && dtype != at::kFloat) throw Decline{};
        m.dtype = dtype == at::kBFloat16 ? KVCOMM_BF16 : KVCOMM_F32;
    }

private:
    struct py {   // owned reference
        PyObject *o;
        explicit py(PyObject *p) : o(p) {}
        py(py &&r) : o(r.o) { r.o = nullptr; }
        ~py() { Py_XDECREF(o); }
    };
};

// [layer, head, token, channel] tensor with contiguous channels
kvcomm_tensor desc(const at::Tensor &t, at::ScalarType dtype)
{
    if (t.scalar_type() != dtype || t.dim() != 4 || t.stride(3) != 1) throw Decline{};
    return kvcomm_tensor{t.data_ptr(), t.stride(0), t.stride(1), t.stride(2)};
}
kvcomm_tensor desc(PyObject *o, at::ScalarType dtype) { return desc(as_tensor(o), dtype); }

bool same_layout(const kvcomm_tensor &a, const kvcomm_tensor &b)
{
    return a.stride_layer == b.stride_layer && a.stride_head == b.stride_head && a.stride_token == b.stride_token;
}

struct Items {   // of a list or tuple
    PyObject *const *p;
    int n;
    Items(PyObject *o, int max, int min = 1)
    {
        if (!PyList_CheckExact(o) && !PyTuple_CheckExact(o)) throw Decline{};
        const Py_ssize_t len = PySequence_Fast_GET_SIZE(o);
        if (len < min || len > max) throw Decline{};
        p = PySequence_Fast_ITEMS(o);
        n = (int)len;
    }
};

void ints(PyObject *o, int n, int32_t *out)
{
    const Items it(o, n);
    if (it.n != n) throw Decline{};
    for (int i = 0; i < n; ++i) out[i] = as_int(it.p[i]);
}

void floats(PyObject *o, int n, float *out)
{
    const Items it(o, n);
    if (it.n != n) throw Decline{};
    for (int i = 0; i < n; ++i) out[i] = (float)as_double(it.p[i]);
}

// Anchors of one layout: pointers, layout, and lengths (those of the tensors where none are given).
struct Anchors {
    const void *ptr[kMaxAnchors];
    int32_t len[kMaxAnchors];
    kvcomm_tensor layout;
    int n;
    void read(PyObject *list, at::ScalarType dtype)
    {
        const Items it(list, kMaxAnchors);
        n = it.n;
        c10::IntArrayRef strides;
        for (int a = 0; a < n; ++a) {
            const at::Tensor &t = as_tensor(it.p[a]);
            if (a == 0) {
                layout = desc(t, dtype);
                strides = t.strides();
            } else if (t.scalar_type() != dtype || t.strides() != strides) {
                throw Decline{};
            }
            ptr[a] = t.data_ptr();
            const int64_t tokens = t.size(2);
            if (tokens > INT32_MAX) throw Decline{};
            len[a] = (int32_t)tokens;
        }
    }
    void lengths(PyObject *o) { if (o != Py_None) ints(o, n, len); }
};

void *data_or_null(PyObject *o) { return o == Py_None ? nullptr : as_tensor(o).data_ptr(); }

const float *weights_of(PyObject *o, int64_t *numel)
{
    const at::Tensor &w = as_tensor(o);
    if (w.scalar_type() != at::kFloat || !w.is_contiguous()) throw Decline{};
    *numel = w.numel();
    return static_cast<const float *>(w.data_ptr());
}

struct Scratch {
    void *ptr = nullptr;
    size_t bytes = 0;
    explicit Scratch(PyObject *o)
    {
        if (o == Py_None) return;
        const at::Tensor &t = as_tensor(o);
        ptr = t.data_ptr();
        bytes = (size_t)t.numel() * t.element_size();
    }
};

int32_t tokens_of(const at::Tensor &t)
{
    if (t.dim() != 4 || t.size(2) > INT32_MAX) throw Decline{};
    return (int32_t)t.size(2);
}

// The stream's handle: the given one's, or the current one's on the current device.
void *stream_of(PyObject *o)
{
    PyObject *h;
    if (o != Py_None) {
        h = PyObject_GetAttr(o, names.cuda_stream);
    } else {
        if (lib.current_stream == Py_None) throw Decline{};
        PyObject *dev = PyObject_CallNoArgs(lib.current_device);
        if (!dev) throw Decline{};
        h = PyObject_CallOneArg(lib.current_stream, dev);
        Py_DECREF(dev);
    }
    if (!h) throw Decline{};
    const unsigned long long v = PyLong_CheckExact(h) ? PyLong_AsUnsignedLongLong(h) : 0;
    const bool ok = PyLong_CheckExact(h) && !PyErr_Occurred();
    Py_DECREF(h);
    if (!ok) throw Decline{};
    return reinterpret_cast<void *>((uintptr_t)v);
}

PyObject *item(PyObject *dict, PyObject *name)   // borrowed; None where there is none
{
    PyObject *v = PyDict_GetItemWithError(dict, name);
    if (!v && PyErr_Occurred()) throw Decline{};
    return v ? v : Py_None;
}

// Runs F over exactly N arguments; whatever is not plain comes back as None.
template <int N, class F>
PyObject *entry(PyObject *const *a, Py_ssize_t n, F &&f)
{
    if (n != N) {
        PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
        return nullptr;
    }
    try {
        return PyLong_FromLongLong(f(a));
    } catch (abi::__forced_unwind &) {   // the thread is being ended (see unlocked())
        throw;
    } catch (...) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
}

// The library's call, without the interpreter lock: a launch waits where the queue is full.  A daemon thread that asks for the lock
// again while the interpreter shuts down is ended there, by an unwinding that no destructor, noexcept or catch may stop.  The
// library itself throws nothing.
template <class F>
long long unlocked(F &&f)
{
    PyThreadState *st = PyEval_SaveThread();
    const long long status = f();
    PyEval_RestoreThread(st);
    return status;
}

// -------------------------------------------------------------------------------------------- entry points
// (model, n_ctx, tq)
PyObject *suffix_attn_workspace(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    return entry<3>(args, n, [](PyObject *const *a) {
        const Call c(a[0]);
        return (long long)lib.attn_workspace(&c.m, as_int(a[1]), as_int(a[2]));
    });
}

// (model, gran, rule, temperature, seg_base_k, anchor_base_k, anchor_len, weights_out, nearest_out, selected_out, workspace, stream)
PyObject *anchor_weights(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    return entry<12>(args, n, [](PyObject *const *a) {
        const Call c(a[0]);
        const int32_t gran = as_int(a[1]), rule = as_int(a[2]);
        const float tau = (float)as_double(a[3]);
        const at::Tensor &seg = as_tensor(a[4]);
        const kvcomm_tensor s = desc(seg, c.dtype);
        const int32_t S = tokens_of(seg);
        Anchors anc;
        anc.read(a[5], c.dtype);
        anc.lengths(a[6]);
        float *w = static_cast<float *>(as_tensor(a[7]).data_ptr());
        int32_t *nearest = static_cast<int32_t *>(as_tensor(a[8]).data_ptr()), *sel = static_cast<int32_t *>(as_tensor(a[9]).data_ptr());
        const Scratch ws(a[10]);
        void *stream = stream_of(a[11]);
        return unlocked([&] {
            return lib.anchor_weights_rule(&c.m, gran, rule, tau, s, S, anc.ptr, anc.layout, anc.len, anc.n, w, nearest, sel, ws.ptr, ws.bytes, stream);
        });
    });
}

// (model, gran, rule, temperature, jobs, outputs of each job as (weights, nearest, selected), workspace, stream)
PyObject *anchor_weights_batch(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    return entry<8>(args, n, [](PyObject *const *a) {
        const Call c(a[0]);
        const int32_t gran = as_int(a[1]), rule = as_int(a[2]);
        const float tau = (float)as_double(a[3]);
        const Items jobs(a[4], kMaxBatch), outs(a[5], kMaxBatch);
        if (outs.n != jobs.n) throw Decline{};
        Anchors anc[kMaxBatch];
        kvcomm_weights_job cj[kMaxBatch];
        for (int j = 0; j < jobs.n; ++j) {
            PyObject *d = jobs.p[j];
            if (!PyDict_CheckExact(d)) throw Decline{};
            const at::Tensor &seg = as_tensor(item(d, names.seg_base_k));
            anc[j].read(item(d, names.anchor_base_k), c.dtype);
            anc[j].lengths(item(d, names.anchor_len));
            if (!same_layout(anc[0].layout, anc[j].layout)) throw Decline{};
            const Items o(outs.p[j], 3);
            if (o.n != 3) throw Decline{};
            cj[j] = kvcomm_weights_job{desc(seg, c.dtype), tokens_of(seg), anc[j].ptr, anc[j].len, anc[j].n,
                                       static_cast<float *>(as_tensor(o.p[0]).data_ptr()),
                                       static_cast<int32_t *>(as_tensor(o.p[1]).data_ptr()),
                                       static_cast<int32_t *>(as_tensor(o.p[2]).data_ptr())};
        }
        const Scratch ws(a[6]);
        void *stream = stream_of(a[7]);
        return unlocked([&] { return lib.anchor_weights_batch(&c.m, gran, rule, tau, anc[0].layout, cj, jobs.n, ws.ptr, ws.bytes, stream); });
    });
}

// What a job of the update has beside its anchors, from the objects in the order of `o`: base_k, base_v, weights, delta_pos,
// anchor_delta_pos, out_k, out_v
template <class Job>
void update_job(const Call &c, PyObject *const (&o)[7], const Anchors &k, const Anchors &v, int32_t *adp, Job &job, int64_t *numel)
{
    if (k.n != v.n || !same_layout(k.layout, v.layout)) throw Decline{};
    const at::Tensor &base = as_tensor(o[0]);
    job.base_k = desc(base, c.dtype);
    job.base_v = desc(o[1], c.dtype);
    job.seg_len = tokens_of(base);
    job.out_k = desc(o[5], c.dtype);
    job.out_v = desc(o[6], c.dtype);
    job.delta_pos = as_int(o[3]);
    job.anchor_dk = k.ptr;
    job.anchor_dv = v.ptr;
    job.anchor_len = k.len;
    job.anchor_delta_pos = nullptr;
    if (o[4] != Py_None) {
        ints(o[4], k.n, adp);
        job.anchor_delta_pos = adp;
    }
    job.n_anchors = k.n;
    job.weights = weights_of(o[2], numel);
}

// (model, gran, base_k, base_v, anchor_dk, anchor_dv, weights, delta_pos, out_k, out_v, anchor_len, anchor_delta_pos, stream)
PyObject *align_kv(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    return entry<13>(args, n, [](PyObject *const *a) {
        const Call c(a[0]);
        const int32_t gran = as_int(a[1]);
        Anchors k, v;
        k.read(a[4], c.dtype);
        k.lengths(a[10]);
        v.read(a[5], c.dtype);
        int32_t adp[kMaxAnchors];
        kvcomm_align_job j;
        int64_t numel;
        update_job(c, {a[2], a[3], a[6], a[7], a[11], a[8], a[9]}, k, v, adp, j, &numel);
        if (numel != (int64_t)(lib.weight_slots(&c.m, j.seg_len, gran) * (size_t)k.n)) throw Decline{};
        void *stream = stream_of(a[12]);
        return unlocked([&] {
            return lib.align_kv(&c.m, gran, j.base_k, j.base_v, j.seg_len, k.ptr, v.ptr, k.layout, k.len, k.n, j.weights, j.delta_pos,
                                j.anchor_delta_pos, j.out_k, j.out_v, stream);
        });
    });
}

// (model, gran, base_k, base_v, anchor_dk8, anchor_dv8, scale_k, scale_v, weights, delta_pos, out_k, out_v, anchor_len, anchor_delta_pos, stream)
PyObject *align_kv_q8(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    return entry<15>(args, n, [](PyObject *const *a) {
        const Call c(a[0]);
        const int32_t gran = as_int(a[1]);
        Anchors k, v;
        k.read(a[4], at::kByte);
        k.lengths(a[12]);
        v.read(a[5], at::kByte);
        float sk[kMaxAnchors], sv[kMaxAnchors];
        floats(a[6], k.n, sk);
        floats(a[7], k.n, sv);
        int32_t adp[kMaxAnchors];
        kvcomm_align_q8_job j;
        int64_t numel;
        update_job(c, {a[2], a[3], a[8], a[9], a[13], a[10], a[11]}, k, v, adp, j, &numel);
        if (numel != (int64_t)(lib.weight_slots(&c.m, j.seg_len, gran) * (size_t)k.n)) throw Decline{};
        void *stream = stream_of(a[14]);
        return unlocked([&] {
            return lib.align_kv_q8(&c.m, gran, j.base_k, j.base_v, j.seg_len, k.ptr, v.ptr, k.layout, k.len, sk, sv, k.n, j.weights,
                                   j.delta_pos, j.anchor_delta_pos, j.out_k, j.out_v, stream);
        });
    });
}

// The batched updates: (model, gran, jobs, units or None, stream)
template <bool Q8>
PyObject *update_batch(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    return entry<5>(args, n, [](PyObject *const *a) {
        const Call c(a[0]);
        const int32_t gran = as_int(a[1]);
        const Items jobs(a[2], kMaxBatch);
        const bool beside = a[3] != Py_None;
        const int32_t units = beside ? as_int(a[3]) : 0;
        Anchors k[kMaxBatch], v[kMaxBatch];
        int32_t adp[kMaxBatch][kMaxAnchors];
        float sk[kMaxBatch][kMaxAnchors], sv[kMaxBatch][kMaxAnchors];
        std::conditional_t<Q8, kvcomm_align_q8_job, kvcomm_align_job> cj[kMaxBatch];
        const at::ScalarType stored = Q8 ? at::kByte : c.dtype;
        for (int j = 0; j < jobs.n; ++j) {
            PyObject *d = jobs.p[j];
            if (!PyDict_CheckExact(d)) throw Decline{};
            k[j].read(item(d, Q8 ? names.anchor_dk8 : names.anchor_dk), stored);
            k[j].lengths(item(d, names.anchor_len));
            v[j].read(item(d, Q8 ? names.anchor_dv8 : names.anchor_dv), stored);
            if (!same_layout(k[0].layout, k[j].layout)) throw Decline{};
            int64_t numel;
            update_job(c, {item(d, names.base_k), item(d, names.base_v), item(d, names.weights), item(d, names.delta_pos),
                           item(d, names.anchor_delta_pos), item(d, names.out_k), item(d, names.out_v)}, k[j], v[j], adp[j], cj[j], &numel);
            if (numel % k[j].n) throw Decline{};
            cj[j].weights_slots = numel / k[j].n;
            if constexpr (Q8) {
                floats(item(d, names.scale_k), k[j].n, sk[j]);
                floats(item(d, names.scale_v), k[j].n, sv[j]);
                cj[j].anchor_scale_k = sk[j];
                cj[j].anchor_scale_v = sv[j];
            }
        }
        void *stream = stream_of(a[4]);
        return unlocked([&] {
            if constexpr (Q8)
                return lib.align_kv_q8_batch(&c.m, gran, k[0].layout, cj, jobs.n, stream);
            else
                return beside ? lib.align_kv_batch_beside(&c.m, gran, k[0].layout, cj, jobs.n, units, stream)
                              : lib.align_kv_batch(&c.m, gran, k[0].layout, cj, jobs.n, stream);
        });
    });
}

// (model, q, cache_k, cache_v, n_ctx, softmax_scale, out, lse_out, max_blocks or None, workspace, stream)
PyObject *suffix_attn(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    return entry<11>(args, n, [](PyObject *const *a) {
        const Call c(a[0]);
        const at::Tensor &q = as_tensor(a[1]);
        const kvcomm_tensor dq = desc(q, c.dtype), dk = desc(a[2], c.dtype), dv = desc(a[3], c.dtype), dout = desc(a[6], c.dtype);
        const int32_t tq = tokens_of(q), n_ctx = as_int(a[4]);
        const float scale = (float)as_double(a[5]);
        float *lse = static_cast<float *>(data_or_null(a[7]));
        const bool confined = a[8] != Py_None;
        const int32_t max_blocks = confined ? as_int(a[8]) : 0;
        const Scratch ws(a[9]);
        void *stream = stream_of(a[10]);
        return unlocked([&] {
            return confined ? lib.suffix_attn_confined_ws(&c.m, dq, dk, dv, n_ctx, tq, scale, dout, lse, max_blocks, ws.ptr, ws.bytes, stream)
                            : lib.suffix_attn(&c.m, dq, dk, dv, n_ctx, tq, scale, dout, lse, ws.ptr, ws.bytes, stream);
        });
    });
}

// (weights, anchor_len, seg_len, gamma, entropy_out, result_out, workspace, stream)
PyObject *anchor_predict(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    return entry<8>(args, n, [](PyObject *const *a) {
        const at::Tensor &w = as_tensor(a[0]);
        if (w.dim() != 2 || w.size(1) < 1 || w.size(1) > kMaxAnchors) throw Decline{};
        int64_t numel;
        const float *wp = weights_of(a[0], &numel);
        const int A = (int)w.size(1);
        int32_t len[kMaxAnchors];
        ints(a[1], A, len);
        const int32_t S = as_int(a[2]);
        const float gamma = (float)as_double(a[3]);
        float *ent = static_cast<float *>(data_or_null(a[4])), *res = static_cast<float *>(as_tensor(a[5]).data_ptr());
        const Scratch ws(a[6]);
        void *stream = stream_of(a[7]);
        return unlocked([&] { return lib.anchor_predict(wp, w.size(0), len, A, S, gamma, ent, res, ws.ptr, ws.bytes, stream); });
    });
}

// (model, base_k, base_v, real_k, real_v, delta_pos, out_dk, out_dv, stream); the shapes have been compared
PyObject *capture_offsets(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    return entry<9>(args, n, [](PyObject *const *a) {
        const Call c(a[0]);
        const at::Tensor &base = as_tensor(a[1]);
        const kvcomm_tensor bk = desc(base, c.dtype), bv = desc(a[2], c.dtype), rk = desc(a[3], c.dtype), rv = desc(a[4], c.dtype),
                            dk = desc(a[6], c.dtype), dv = desc(a[7], c.dtype);
        const int32_t S = tokens_of(base), delta = as_int(a[5]);
        void *stream = stream_of(a[8]);
        return unlocked([&] { return lib.capture_offsets(&c.m, bk, bv, rk, rv, S, delta, dk, dv, stream); });
    });
}

// (model, x, scale, out, stream)
PyObject *quantize_deltas(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    return entry<5>(args, n, [](PyObject *const *a) {
        const Call c(a[0]);
        const at::Tensor &x = as_tensor(a[1]);
        const kvcomm_tensor dx = desc(x, c.dtype), out = desc(a[3], at::kByte);
        const int32_t S = tokens_of(x);
        const float scale = (float)as_double(a[2]);
        void *stream = stream_of(a[4]);
        return unlocked([&] { return lib.quantize_deltas(&c.m, dx, S, scale, out, stream); });
    });
}

// (tensors a, lists of tensors b, tensors c): 1 if no tensor of b or c comes near a byte of a tensor of a and those of c not near
// each other, else 0
PyObject *apart(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    struct Range {
        uintptr_t lo, hi;
        explicit Range(const at::Tensor &t)
        {
            int64_t last = 0;
            for (int64_t d = 0; d < t.dim(); ++d) last += std::max<int64_t>(0, t.size(d) - 1) * t.stride(d);
            lo = reinterpret_cast<uintptr_t>(t.data_ptr());
            hi = lo + (uintptr_t)(last + 1) * t.element_size();
        }
    };
    return entry<3>(args, n, [](PyObject *const *a) {
        const Items own(a[0], INT_MAX, 0), groups(a[1], INT_MAX, 0), each(a[2], INT_MAX, 0);
        std::vector<Range> r;
        auto meets = [&](const Range &o, size_t from, size_t to) {
            return std::any_of(r.begin() + from, r.begin() + to, [&](const Range &x) { return x.lo < o.hi && o.lo < x.hi; });
        };
        for (int i = 0; i < own.n; ++i) r.emplace_back(as_tensor(own.p[i]));
        for (int g = 0; g < groups.n; ++g) {
            const Items other(groups.p[g], INT_MAX, 0);
            for (int k = 0; k < other.n; ++k)
                if (meets(Range(as_tensor(other.p[k])), 0, own.n)) return 0LL;
        }
        for (int i = 0; i < each.n; ++i) {
            r.emplace_back(as_tensor(each.p[i]));
            if (meets(r.back(), 0, r.size() - 1)) return 0LL;
        }
        return 1LL;
    });
}

// bind(addresses by entry point's name, Model, current_device, current_stream or None)
PyObject *bind(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (n != 4 || !PyDict_CheckExact(a[0])) {
        PyErr_SetString(PyExc_TypeError, "bind(dict, Model, current_device, current_stream)");
        return nullptr;
    }
    auto set = [&](auto &fn, const char *name) {
        PyObject *v = PyDict_GetItemString(a[0], name);
        if (!v) return false;
        fn = reinterpret_cast<std::remove_reference_t<decltype(fn)>>((uintptr_t)PyLong_AsUnsignedLongLong(v));
        return !PyErr_Occurred();
    };
    if (!set(lib.weight_slots, "kvcomm_weight_slots") || !set(lib.attn_workspace, "kvcomm_suffix_attn_workspace") ||
        !set(lib.anchor_weights_rule, "kvcomm_anchor_weights_rule") || !set(lib.anchor_weights_batch, "kvcomm_anchor_weights_batch") ||
        !set(lib.align_kv_batch, "kvcomm_align_kv_batch") || !set(lib.align_kv_batch_beside, "kvcomm_align_kv_batch_beside") ||
        !set(lib.align_kv_q8_batch, "kvcomm_align_kv_q8_batch") ||
        !set(lib.align_kv, "kvcomm_align_kv") || !set(lib.align_kv_q8, "kvcomm_align_kv_q8") ||
        !set(lib.suffix_attn, "kvcomm_suffix_attn") || !set(lib.suffix_attn_confined_ws, "kvcomm_suffix_attn_confined_ws") ||
        !set(lib.anchor_predict, "kvcomm_anchor_predict") || !set(lib.capture_offsets, "kvcomm_capture_offsets") ||
        !set(lib.quantize_deltas, "kvcomm_quantize_deltas")) {
        if (!PyErr_Occurred()) PyErr_SetString(PyExc_KeyError, "an entry point of the library is missing");
        return nullptr;
    }
    for (int i = 1; i < 4; ++i) Py_INCREF(a[i]);   // kept until the process ends
    lib.model_type = a[1];
    lib.current_device = a[2];
    lib.current_stream = a[3];
    Py_RETURN_NONE;
}

#define FAST(name, fn) {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(fn)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {FAST("bind", bind),
                         FAST("suffix_attn_workspace", suffix_attn_workspace),
                         FAST("anchor_weights", anchor_weights),
                         FAST("anchor_weights_batch", anchor_weights_batch),
                         FAST("align_kv", align_kv),
                         FAST("align_kv_q8", align_kv_q8),
                         FAST("align_kv_batch", update_batch<false>),
                         FAST("align_kv_q8_batch", update_batch<true>),
                         FAST("suffix_attn", suffix_attn),
                         FAST("anchor_predict", anchor_predict),
                         FAST("capture_offsets", capture_offsets),
                         FAST("quantize_deltas", quantize_deltas),
                         FAST("apart", apart),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal(void)
{
#define NAME(x) \
    if (!(names.x = PyUnicode_InternFromString(#x))) return nullptr
    NAME(n_layers); NAME(n_kv_heads); NAME(n_q_heads); NAME(head_dim); NAME(dtype); NAME(rope_theta); NAME(cuda_stream);
    NAME(seg_base_k); NAME(anchor_base_k); NAME(anchor_len); NAME(base_k); NAME(base_v); NAME(anchor_dk); NAME(anchor_dv);
    NAME(anchor_dk8); NAME(anchor_dv8); NAME(scale_k); NAME(scale_v); NAME(weights); NAME(delta_pos); NAME(anchor_delta_pos);
    NAME(out_k); NAME(out_v);
#undef NAME
    PyObject *m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "built_for", KVC_BUILT_FOR) < 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
