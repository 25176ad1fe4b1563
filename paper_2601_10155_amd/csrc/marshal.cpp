// Marshalling of the per-layer and per-block calls in native code.  The Python functions of binding.py read a dozen
// attributes of every tensor, build a ctypes structure and convert a dozen arguments: 8.5 us a call, more than most decode
// kernels take.  The functions here take the same objects, and where everything is as the call expects it (plain CUDA
// tensors of the right type, shape and layout, output given) they make the library call and return its
// status; where the library chooses the ranges they allocate a missing output and workspace too, and return the output.  Anything else (a copy to make, a buffer to allocate, an argument to refuse) returns None and is left to the Python
// function, so what a call accepts, and with which error it refuses, is written down there alone.
// The entry points are those of the library that binding.py has loaded, handed over as addresses.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <torch/csrc/autograd/python_variable.h>

#include <algorithm>

#include "lookat.h"

namespace {

struct Entries {
    decltype(&lookat_encode_keys) encode_keys;
    decltype(&lookat_build_lut) build_lut;
    decltype(&lookat_attend_decode) attend_decode;
    decltype(&lookat_attend_decode_workspace_bytes) attend_decode_workspace_bytes;
    decltype(&lookat_decode_step) decode_step;
    decltype(&lookat_decode_step_split) decode_step_split;
    decltype(&lookat_decode_step_split_workspace_bytes) decode_step_split_workspace_bytes;
    decltype(&lookat_decode_step_gqa) decode_step_gqa;
    decltype(&lookat_decode_step_gqa_workspace_bytes) decode_step_gqa_workspace_bytes;
    decltype(&lookat_score_prefill) score_prefill;
};
Entries entry = {};
PyObject *stream_of_device = nullptr;   // torch's "current raw stream of device i"

// A tensor whose memory can be handed to the library as it is (no subclass, no wrapper of a transform), or nullptr.
const at::Tensor *plain(PyObject *o)
{
    if (!THPVariable_CheckTypeExact(Py_TYPE(o)))
        return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.defined() || !t.is_cuda() || t.layout() != at::kStrided || !t.has_storage() || t.is_neg() || t.is_conj() || t.numel() == 0)
        return nullptr;
    return &t;
}
const at::Tensor *plain(PyObject *o, at::ScalarType dtype)
{
    const at::Tensor *t = plain(o);
    return t && t->scalar_type() == dtype ? t : nullptr;
}
const at::Tensor *dense(PyObject *o, at::ScalarType dtype)
{
    const at::Tensor *t = plain(o, dtype);
    return t && t->is_contiguous() ? t : nullptr;
}
// fp16 or fp32, dense
const at::Tensor *dense_float(PyObject *o, lookat_dtype &tag)
{
    const at::Tensor *t = plain(o);
    if (!t || !t->is_contiguous())
        return nullptr;
    if (t->scalar_type() == at::kHalf)
        tag = LOOKAT_F16;
    else if (t->scalar_type() == at::kFloat)
        tag = LOOKAT_F32;
    else
        return nullptr;
    return t;
}

// Element stride between the (b,h) slabs of a [B,H,L,X] tensor whose slabs are dense.
bool bh_stride(const at::Tensor &t, int64_t &stride)
{
    const int64_t B = t.size(0), H = t.size(1), L = t.size(2), X = t.size(3);
    if (t.stride(3) != 1 || (L > 1 && t.stride(2) != X))
        return false;
    stride = H > 1 ? t.stride(1) : std::max(t.stride(0), L * X);
    return B == 1 || t.stride(0) == H * stride;
}

bool number(PyObject *o, float &v)
{
    const double d = PyFloat_AsDouble(o);
    if (d == -1.0 && PyErr_Occurred()) {
        PyErr_Clear();
        return false;
    }
    v = (float)d;
    return true;
}
bool integer(PyObject *o, int64_t low, int64_t high, int64_t &v)
{
    if (!PyLong_CheckExact(o))
        return false;
    int overflow = 0;
    const long long x = PyLong_AsLongLongAndOverflow(o, &overflow);
    v = x;
    return !overflow && x >= low && x <= high;
}

bool current_stream(const at::Tensor &t, void *&stream)
{
    PyObject *index = PyLong_FromLong(t.device().index());
    PyObject *s = index ? PyObject_CallFunctionObjArgs(stream_of_device, index, nullptr) : nullptr;
    Py_XDECREF(index);
    if (!s) {
        PyErr_Clear();
        return false;
    }
    stream = PyLong_AsVoidPtr(s);
    Py_DECREF(s);
    if (PyErr_Occurred()) {
        PyErr_Clear();
        return false;
    }
    return true;
}

bool shape_of(int64_t B, int64_t H, int64_t d_k, int64_t m, lookat_shape &s)
{
    if (B <= 0 || H <= 0 || d_k <= 0 || m <= 0 || std::max({B, H, d_k, m}) > 0x7fffffff)
        return false;
    s = lookat_shape{(int32_t)B, (int32_t)H, (int32_t)d_k, (int32_t)m, 256};
    return true;
}

PyObject *status(int rc) { return PyLong_FromLong(rc); }

#define GIVE_UP Py_RETURN_NONE
// The GIL is released while the library enqueues, as ctypes does.
#define CALL(rc_, expr_)          \
    int rc_;                      \
    Py_BEGIN_ALLOW_THREADS rc_ = (expr_); \
    Py_END_ALLOW_THREADS

// codebooks [H, m, 256, d_k / m] fp32, dense
const at::Tensor *codebooks_of(PyObject *o)
{
    const at::Tensor *cb = dense(o, at::kFloat);
    return cb && cb->dim() == 4 && cb->size(2) == 256 ? cb : nullptr;
}

// (workspace object, bytes needed) -> pointer and size as binding.py would pass them; false: left to it.
// `choice`: the ranges are the library's choice.  No workspace is then allocated here (`own`; on the current stream of that device, the
// one the library is given, and returned to the allocator in its order): the Python path's allocation and second look
// at the arguments cost as much as the ranges save (12 heads x 1024 keys, d_k = 128, attention without a workspace: 14.3 us a call;
// 8.9 before the library cut such contexts; 6.9 now).
// `fits`: the library takes fewer ranges where a given workspace does not hold its choice (or refuses, see answer()).
bool workspace_of(PyObject *o, size_t need, bool choice, bool fits, const at::Tensor &like, at::Tensor &own, void *&ptr, size_t &bytes)
{
    ptr = nullptr;
    bytes = 0;
    if (o == Py_None) {
        if (need && choice) {
            own = at::empty({(int64_t)need}, like.options().dtype(at::kByte));
            ptr = own.data_ptr();
            bytes = need;
        }
        return need == 0 || choice;
    }
    const at::Tensor *w = plain(o);
    if (!w)
        return false;
    ptr = w->data_ptr();
    bytes = (size_t)w->numel() * w->element_size();
    return fits || bytes >= need;
}
// A workspace that the library refuses is too small even for that: one has to be allocated.
PyObject *answer(int rc)
{
    if (rc == LOOKAT_ERR_WORKSPACE)
        GIVE_UP;
    return status(rc);
}

// The result of a call that was given no `out`: the tensor, or the status where that is not LOOKAT_OK.
PyObject *answer(int rc, at::Tensor &made)
{
    return rc == LOOKAT_OK && made.defined() ? THPVariable_Wrap(std::move(made)) : answer(rc);
}

// q, k_new, codebooks, codes, values, scale, [num_splits, workspace,] out: kind 0 decode_step, 1 split, 2 gqa
PyObject *step(PyObject *const *args, Py_ssize_t n, int kind)
{
    if (n != (kind ? 9 : 7))
        GIVE_UP;
    PyObject *out_o = args[n - 1];
    lookat_dtype qt, kt;
    const at::Tensor *q = dense_float(args[0], qt), *k = dense_float(args[1], kt), *cb = codebooks_of(args[2]);
    const at::Tensor *codes = plain(args[3], at::kByte), *values = plain(args[4], at::kHalf), *out = nullptr;
    if (out_o != Py_None || !kind) {
        out = dense(out_o, at::kFloat);
        if (!out)
            GIVE_UP;
    }
    float scale;
    int64_t splits = 0, cs, vs;
    if (!q || !k || !cb || !codes || !values || qt != kt || codes->dim() != 4 || values->dim() != 4 || !number(args[5], scale) ||
        (kind && !integer(args[6], 0, 0x7fffffff, splits)))
        GIVE_UP;
    const int64_t B = codes->size(0), H = codes->size(1), L = codes->size(2), m = codes->size(3), d_k = values->size(3);
    lookat_shape s;
    if (!shape_of(B, H, d_k, m, s) || values->size(0) != B || values->size(1) != H || values->size(2) != L || d_k % m ||
        cb->size(0) != H || cb->size(1) != m || cb->size(3) != d_k / m || k->numel() != B * H * d_k || !bh_stride(*codes, cs) ||
        !bh_stride(*values, vs))
        GIVE_UP;
    int64_t group = 1;
    if (kind == 2) {
        if (q->dim() != 3 || q->size(0) != B || q->size(1) % H || q->size(2) != d_k)
            GIVE_UP;
        group = q->size(1) / H;
        if (group > 0x7fffffff)
            GIVE_UP;
    } else if (q->numel() != B * H * d_k) {
        GIVE_UP;
    }
    if (out ? out->numel() != B * H * group * d_k : splits != 0)
        GIVE_UP;
    void *ws = nullptr, *stream;
    size_t ws_bytes = 0;
    at::Tensor own;
    if (kind) {
        const size_t need = kind == 1 ? entry.decode_step_split_workspace_bytes(&s, L, (int32_t)splits)
                                      : entry.decode_step_gqa_workspace_bytes(&s, (int32_t)group, L, (int32_t)splits);
        if (!workspace_of(args[7], need, splits == 0, splits == 0 && group == 1, *values, own, ws, ws_bytes))
            GIVE_UP;
    }
    if (!current_stream(*values, stream))
        GIVE_UP;
    const float *cbp = static_cast<const float *>(cb->data_ptr());
    uint8_t *cp = static_cast<uint8_t *>(codes->data_ptr());
    at::Tensor made;
    if (!out)
        made = at::empty({B, H * group, d_k}, values->options().dtype(at::kFloat));
    float *op = static_cast<float *>((out ? *out : made).data_ptr());
    const void *qp = q->data_ptr(), *kp = k->data_ptr(), *vp = values->data_ptr();
    CALL(rc, kind == 0   ? entry.decode_step(&s, L, qp, kp, qt, cbp, cp, cs, vp, vs, scale, op, stream)
             : kind == 1 ? entry.decode_step_split(&s, L, qp, kp, qt, cbp, cp, cs, vp, vs, scale, (int32_t)splits, ws, ws_bytes, op, stream)
                         : entry.decode_step_gqa(&s, (int32_t)group, L, qp, kp, qt, cbp, cp, cs, vp, vs, scale, (int32_t)splits, ws,
                                                 ws_bytes, op, stream));
    return answer(rc, made);
}

// lut, codes, values, scale, num_splits, workspace, out, scores_out
PyObject *attend(PyObject *const *args, Py_ssize_t n)
{
    if (n != 8)
        GIVE_UP;
    const at::Tensor *lut = dense(args[0], at::kFloat), *codes = plain(args[1], at::kByte), *values = plain(args[2], at::kHalf);
    const at::Tensor *out = args[6] == Py_None ? nullptr : dense(args[6], at::kFloat), *scores = args[7] == Py_None ? nullptr : dense(args[7], at::kFloat);
    float scale;
    int64_t splits, cs, vs;
    if (!lut || !codes || !values || (args[6] != Py_None && !out) || (args[7] != Py_None && !scores) || codes->dim() != 4 || values->dim() != 4 ||
        !number(args[3], scale) || !integer(args[4], 0, 0x7fffffff, splits))
        GIVE_UP;
    const int64_t B = codes->size(0), H = codes->size(1), L = codes->size(2), m = codes->size(3), d_k = values->size(3);
    lookat_shape s;
    if (!shape_of(B, H, d_k, m, s) || values->size(0) != B || values->size(1) != H || values->size(2) != L ||
        lut->numel() != B * H * m * 256 || (out ? out->numel() != B * H * d_k : splits != 0) || (scores && scores->numel() != B * H * L) ||
        !bh_stride(*codes, cs) || !bh_stride(*values, vs))
        GIVE_UP;
    void *ws, *stream;
    size_t ws_bytes;
    at::Tensor own;
    if (!workspace_of(args[5], entry.attend_decode_workspace_bytes(&s, L, (int32_t)splits), splits == 0, splits == 0, *values, own, ws,
                      ws_bytes) ||
        !current_stream(*values, stream))
        GIVE_UP;
    at::Tensor made;
    if (!out)
        made = at::empty({B, H, d_k}, values->options().dtype(at::kFloat));
    float *op = static_cast<float *>((out ? *out : made).data_ptr());
    CALL(rc, entry.attend_decode(&s, L, static_cast<const float *>(lut->data_ptr()), static_cast<const uint8_t *>(codes->data_ptr()), cs,
                                 values->data_ptr(), vs, scale, (int32_t)splits, ws, ws_bytes, op,
                                 scores ? static_cast<float *>(scores->data_ptr()) : nullptr, stream));
    return answer(rc, made);
}

// keys, codebooks, codes_out | None, cache | None, position
PyObject *encode(PyObject *const *args, Py_ssize_t n)
{
    if (n != 5)
        GIVE_UP;
    lookat_dtype kt;
    const at::Tensor *keys = dense_float(args[0], kt), *cb = codebooks_of(args[1]);
    int64_t position;
    if (!keys || !cb || keys->dim() != 4 || !integer(args[4], 0, INT64_MAX, position))
        GIVE_UP;
    const int64_t B = keys->size(0), H = keys->size(1), N = keys->size(2), d_k = keys->size(3), m = cb->size(1);
    lookat_shape s;
    if (!shape_of(B, H, d_k, m, s) || cb->size(0) != H || m * cb->size(3) != d_k)
        GIVE_UP;
    uint8_t *dst;
    int64_t stride;
    if (args[3] != Py_None) {
        const at::Tensor *cache = plain(args[3], at::kByte);
        if (!cache || cache->dim() != 4 || cache->size(0) != B || cache->size(1) != H || cache->size(3) != m || N > cache->size(2) ||
            position > cache->size(2) - N || !bh_stride(*cache, stride))
            GIVE_UP;
        dst = static_cast<uint8_t *>(cache->data_ptr()) + position * m;
    } else {
        const at::Tensor *codes = dense(args[2], at::kByte);
        if (!codes || codes->dim() != 4 || codes->size(0) != B || codes->size(1) != H || codes->size(2) != N || codes->size(3) != m)
            GIVE_UP;
        dst = static_cast<uint8_t *>(codes->data_ptr());
        stride = N * m;
    }
    void *stream;
    if (!current_stream(*keys, stream))
        GIVE_UP;
    CALL(rc, entry.encode_keys(&s, N, keys->data_ptr(), kt, static_cast<const float *>(cb->data_ptr()), dst, stride, stream));
    return status(rc);
}

// q, codebooks, lut_out
PyObject *lut(PyObject *const *args, Py_ssize_t n)
{
    if (n != 3)
        GIVE_UP;
    lookat_dtype qt;
    const at::Tensor *q = dense_float(args[0], qt), *cb = codebooks_of(args[1]), *out = dense(args[2], at::kFloat);
    if (!q || !cb || !out || q->dim() != 4)
        GIVE_UP;
    const int64_t B = q->size(0), H = q->size(1), T = q->size(2), d_k = q->size(3), m = cb->size(1);
    lookat_shape s;
    void *stream;
    if (!shape_of(B, H, d_k, m, s) || T > 0x7fffffff || cb->size(0) != H || m * cb->size(3) != d_k || out->numel() != B * H * T * m * 256 ||
        !current_stream(*q, stream))
        GIVE_UP;
    CALL(rc, entry.build_lut(&s, (int32_t)T, q->data_ptr(), qt, static_cast<const float *>(cb->data_ptr()),
                             static_cast<float *>(out->data_ptr()), stream));
    return status(rc);
}

// q, codebooks, codes, scores_out
PyObject *prefill(PyObject *const *args, Py_ssize_t n)
{
    if (n != 4)
        GIVE_UP;
    lookat_dtype qt;
    int64_t cs;
    const at::Tensor *q = dense_float(args[0], qt), *cb = codebooks_of(args[1]), *codes = plain(args[2], at::kByte);
    const at::Tensor *out = dense(args[3], at::kFloat);
    if (!q || !cb || !codes || !out || q->dim() != 4 || codes->dim() != 4)
        GIVE_UP;
    const int64_t B = q->size(0), H = q->size(1), T = q->size(2), d_k = q->size(3), m = cb->size(1), L = codes->size(2);
    lookat_shape s;
    void *stream;
    if (!shape_of(B, H, d_k, m, s) || T > 0x7fffffff || cb->size(0) != H || m * cb->size(3) != d_k || codes->size(0) != B ||
        codes->size(1) != H || codes->size(3) != m || out->numel() != B * H * T * L || !bh_stride(*codes, cs) || !current_stream(*q, stream))
        GIVE_UP;
    CALL(rc, entry.score_prefill(&s, (int32_t)T, L, q->data_ptr(), qt, static_cast<const float *>(cb->data_ptr()),
                                 static_cast<const uint8_t *>(codes->data_ptr()), cs, static_cast<float *>(out->data_ptr()), stream));
    return status(rc);
}

// No C++ exception crosses into the interpreter: whatever torch throws while a tensor is looked at, the Python function
// will meet as well, and raise.
template <PyObject *(*F)(PyObject *const *, Py_ssize_t)>
PyObject *guarded(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    if (!entry.score_prefill)
        GIVE_UP;
    try {
        return F(args, n);
    } catch (...) {
        GIVE_UP;
    }
}
PyObject *step0(PyObject *const *a, Py_ssize_t n) { return step(a, n, 0); }
PyObject *step1(PyObject *const *a, Py_ssize_t n) { return step(a, n, 1); }
PyObject *step2(PyObject *const *a, Py_ssize_t n) { return step(a, n, 2); }

// bind(current_raw_stream, addresses of the entry points in the order of Entries)
PyObject *bind(PyObject *, PyObject *args)
{
    PyObject *fn;
    unsigned long long a[10];
    if (!PyArg_ParseTuple(args, "OKKKKKKKKKK", &fn, a, a + 1, a + 2, a + 3, a + 4, a + 5, a + 6, a + 7, a + 8, a + 9))
        return nullptr;
    Py_INCREF(fn);
    Py_XDECREF(stream_of_device);
    stream_of_device = fn;
    entry.encode_keys = reinterpret_cast<decltype(entry.encode_keys)>(a[0]);
    entry.build_lut = reinterpret_cast<decltype(entry.build_lut)>(a[1]);
    entry.attend_decode = reinterpret_cast<decltype(entry.attend_decode)>(a[2]);
    entry.attend_decode_workspace_bytes = reinterpret_cast<decltype(entry.attend_decode_workspace_bytes)>(a[3]);
    entry.decode_step = reinterpret_cast<decltype(entry.decode_step)>(a[4]);
    entry.decode_step_split = reinterpret_cast<decltype(entry.decode_step_split)>(a[5]);
    entry.decode_step_split_workspace_bytes = reinterpret_cast<decltype(entry.decode_step_split_workspace_bytes)>(a[6]);
    entry.decode_step_gqa = reinterpret_cast<decltype(entry.decode_step_gqa)>(a[7]);
    entry.decode_step_gqa_workspace_bytes = reinterpret_cast<decltype(entry.decode_step_gqa_workspace_bytes)>(a[8]);
    entry.score_prefill = reinterpret_cast<decltype(entry.score_prefill)>(a[9]);
    Py_RETURN_NONE;
}

template <PyObject *(*F)(PyObject *const *, Py_ssize_t)>
PyMethodDef method(const char *name)
{
    return PyMethodDef{name, (PyCFunction)(void (*)(void))guarded<F>, METH_FASTCALL, nullptr};
}
PyMethodDef methods[] = {method<step0>("decode_step"),   method<step1>("decode_step_split"), method<step2>("decode_step_gqa"),
                         method<attend>("attend_decode"), method<encode>("encode_keys"),      method<lut>("build_lut"),
                         method<prefill>("score_prefill"), {"bind", bind, METH_VARARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal(void) { return PyModule_Create(&module); }
