// CPython binding of the C ABI (include/slimattn.h): checks torch tensors, allocates the results a caller leaves out,
// takes the current HIP stream and calls.  slimattn.py holds the public signatures and hands its arguments over.
//
// What a small call costs is its launches (2.4 us of host time each, most of it the runtime's hand-over of the
// kernel arguments) plus this marshalling.  Done in Python with ctypes the marshalling took 5 to 7 us a call
// (torch.cuda.current_stream() 2.7, eight attribute reads and a ctypes pointer per tensor 0.7 each), more than the
// launch; here it takes well under 1 us.
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <c10/core/DefaultDtype.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <algorithm>

#include "../../include/slimattn.h"

namespace {

PyObject* g_raise_status = nullptr;   // slimattn._check: turns a status into SlimError

struct Failed {};   // a Python error is set

[[noreturn]] void fail(PyObject* type, const char* text) {
    PyErr_SetString(type, text);
    throw Failed();
}
inline void require(bool ok, const char* text) {
    if (__builtin_expect(!ok, 0)) fail(PyExc_AssertionError, text);
}

const at::Tensor& tensor(PyObject* o) {
    if (!THPVariable_Check(o)) fail(PyExc_TypeError, "expected a torch tensor");
    return THPVariable_Unpack(o);
}
inline bool given(PyObject* o) { return o != Py_None; }

// Device address of a densely packed device tensor.
void* ptr(const at::Tensor& t) {
    require(t.is_cuda() && t.is_contiguous(), "device tensors, densely packed");
    return t.data_ptr();
}
void* ptr(const at::Tensor& t, at::ScalarType dtype, const char* text) {
    require(t.is_cuda() && t.is_contiguous(), "device tensors, densely packed");
    require(t.scalar_type() == dtype, text);
    return t.data_ptr();
}
void* bf16_ptr(const at::Tensor& t) { return ptr(t, at::kBFloat16, "expected torch.bfloat16"); }
int8_t* i8_ptr(const at::Tensor& t) { return (int8_t*)ptr(t, at::kChar, "expected torch.int8"); }
float* f32_ptr(const at::Tensor& t) { return (float*)ptr(t, at::kFloat, "expected torch.float32"); }
int32_t* i32_ptr(const at::Tensor& t) { return (int32_t*)ptr(t, at::kInt, "expected torch.int32"); }

inline void require_shape(const at::Tensor& t, std::initializer_list<int64_t> want, const char* text) {
    const at::IntArrayRef s = t.sizes();
    require(s.size() == want.size() && std::equal(s.begin(), s.end(), want.begin()), text);
}

// A result the caller passes is written densely from its first element: it has to hold all of it (its shape is the
// caller's affair: a flat buffer, or one that has room for more, will do).
inline void require_room(const at::Tensor& t, int64_t n, const char* text) { require(t.numel() >= n, text); }

struct Dims4 {
    int64_t b, h, s, d;
    int64_t rows() const { return b * h * s; }
    int64_t count() const { return rows() * d; }
};
Dims4 dims4(const at::Tensor& t) {
    if (t.dim() != 4) fail(PyExc_ValueError, "expected a tensor of four dimensions");
    const auto s = t.sizes();
    return {s[0], s[1], s[2], s[3]};
}
// Sizes reach the library as C ints; one that does not fit is passed on as 0, which the library refuses.
inline int c_int(int64_t v) { return v >= 0 && v <= 0x7fffffff ? (int)v : 0; }

// Lets other Python threads run: an allocation may have to wait for the device.
struct WithoutInterpreterLock {
    PyThreadState* const state = PyEval_SaveThread();
    ~WithoutInterpreterLock() { PyEval_RestoreThread(state); }
};

at::Tensor make(std::initializer_list<int64_t> shape, at::ScalarType dtype, const at::Tensor& like) {
    const WithoutInterpreterLock unlocked;
    return at::empty(at::IntArrayRef(shape.begin(), shape.size()), like.options().dtype(dtype).requires_grad(false));
}

float as_float(PyObject* o) {
    const double v = PyFloat_AsDouble(o);
    if (v == -1.0 && PyErr_Occurred()) throw Failed();
    return (float)v;
}
int as_flag(PyObject* o) {
    const int v = PyObject_IsTrue(o);
    if (v < 0) throw Failed();
    return v;
}
// The result's type; None is torch's default type, as for torch.empty
at::ScalarType out_type(PyObject* o) {
    if (!given(o)) return c10::typeMetaToScalarType(c10::get_default_dtype());
    if (!THPDtype_Check(o)) fail(PyExc_TypeError, "out_dtype must be a torch.dtype");
    return reinterpret_cast<THPDtype*>(o)->scalar_type;
}

// The C call runs without the interpreter lock (a full hardware queue makes a launch wait); a status other than
// SLIM_OK becomes the Python exception.
template <class F>
void call(F&& f) {
    const hipStream_t stream = c10::hip::getCurrentHIPStream().stream();
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = f((void*)stream);
    Py_END_ALLOW_THREADS
    if (__builtin_expect(status != SLIM_OK, 0)) {
        PyObject* r = PyObject_CallFunction(g_raise_status, "i", status);
        Py_XDECREF(r);
        if (r != nullptr) PyErr_SetString(PyExc_RuntimeError, "the library reported a failed call");
        throw Failed();
    }
}

// Optional output: the caller's tensor, or a new one.
at::Tensor out_or_new(PyObject* o, std::initializer_list<int64_t> shape, at::ScalarType dtype, const at::Tensor& like) {
    return given(o) ? tensor(o) : make(shape, dtype, like);
}

PyObject* wrap(const at::Tensor& t) { return THPVariable_Wrap(t); }
PyObject* give(PyObject* passed, const at::Tensor& t) {   // the very object the caller passed, where there is one
    if (given(passed)) {
        Py_INCREF(passed);
        return passed;
    }
    return wrap(t);
}
template <size_t N>
PyObject* tuple_of(PyObject* (&items)[N]) {
    PyObject* t = PyTuple_New(N);
    for (size_t i = 0; i < N; ++i) {
        if (t != nullptr && items[i] != nullptr) PyTuple_SET_ITEM(t, i, items[i]);
        else throw Failed();
    }
    return t;
}

typedef PyObject* const* Args;

// x, codes, scales
PyObject* kv_quant(Args a) {
    const at::Tensor& x = tensor(a[0]);
    const Dims4 n = dims4(x);
    const at::Tensor codes = out_or_new(a[1], {n.b, n.h, n.s, n.d}, at::kChar, x);
    const at::Tensor scales = out_or_new(a[2], {n.b, n.h, n.s}, at::kFloat, x);
    require_room(codes, n.count(), "codes is too small");
    require_room(scales, n.rows(), "scales is too small");
    void* const xp = bf16_ptr(x);
    int8_t* const cp = i8_ptr(codes);
    float* const sp = f32_ptr(scales);
    call([&](void* stream) {
        return kv_quant_int8(xp, cp, sp, c_int(n.b), c_int(n.h), c_int(n.h), c_int(n.s), c_int(n.d), 0, 1.0f, stream);
    });
    PyObject* items[2] = {give(a[1], codes), give(a[2], scales)};
    return tuple_of(items);
}

// k, v, k_codes, k_scale, v_codes, v_scale
PyObject* kv_quant_pair(Args a) {
    const at::Tensor &k = tensor(a[0]), &v = tensor(a[1]);
    const Dims4 n = dims4(k);
    require(v.sizes() == k.sizes(), "k and v have one shape");
    at::Tensor codes[2], scales[2];
    for (int i = 0; i < 2; ++i) {
        codes[i] = out_or_new(a[2 + 2 * i], {n.b, n.h, n.s, n.d}, at::kChar, k);
        scales[i] = out_or_new(a[3 + 2 * i], {n.b, n.h, n.s}, at::kFloat, k);
        require_shape(codes[i], {n.b, n.h, n.s, n.d}, "shape of the codes");
        require_shape(scales[i], {n.b, n.h, n.s}, "shape of the scales");
    }
    void *const kp = bf16_ptr(k), *const vp = bf16_ptr(v);
    int8_t *const kc = i8_ptr(codes[0]), *const vc = i8_ptr(codes[1]);
    float *const ks = f32_ptr(scales[0]), *const vs = f32_ptr(scales[1]);
    call([&](void* stream) {
        return kv_quant_int8_pair(kp, vp, kc, ks, vc, vs, c_int(n.b), c_int(n.h), c_int(n.h), c_int(n.s), c_int(n.d), 0, 1.0f, stream);
    });
    PyObject* items[4] = {give(a[2], codes[0]), give(a[3], scales[0]), give(a[4], codes[1]), give(a[5], scales[1])};
    return tuple_of(items);
}

// x_new, codes, scales, positions
PyObject* kv_quant_append(Args a) {
    const at::Tensor &x = tensor(a[0]), &codes = tensor(a[1]), &scales = tensor(a[2]), &positions = tensor(a[3]);
    const Dims4 n = dims4(x), c = dims4(codes);
    require(n.s == 1, "one new token per sequence");
    require_shape(codes, {n.b, n.h, c.s, n.d}, "shape of the codes");
    require_shape(scales, {n.b, n.h, c.s}, "shape of the scales");
    require_shape(positions, {n.b}, "one position per sequence");
    void* const xp = bf16_ptr(x);
    int8_t* const cp = i8_ptr(codes);
    float* const sp = f32_ptr(scales);
    int32_t* const pp = i32_ptr(positions);
    call([&](void* stream) {
        return kv_quant_int8_append(xp, cp, sp, pp, c_int(n.b), c_int(n.h), c_int(n.h), c_int(c.s), c_int(n.d), 0, 1.0f, stream);
    });
    Py_RETURN_NONE;
}

// The result tensor of a prefill: [B, Hq, S, D], bf16 or fp32
at::Tensor prefill_out(PyObject* out, PyObject* dtype, const Dims4& n, const at::Tensor& q) {
    const at::ScalarType t = given(out) ? tensor(out).scalar_type() : out_type(dtype);
    require(t == at::kBFloat16 || t == at::kFloat, "out is bf16 or fp32");
    const at::Tensor o = given(out) ? tensor(out) : make({n.b, n.h, n.s, n.d}, t, q);
    require_room(o, n.count(), "out is too small");
    return o;
}
int out_code(const at::Tensor& o) { return o.scalar_type() == at::kFloat ? SLIM_F32 : SLIM_BF16; }

// q, k, v, softmax_scale, causal, k_scale, v_scale, out, out_dtype
PyObject* prefill(Args a) {
    const at::Tensor &q = tensor(a[0]), &k = tensor(a[1]), &v = tensor(a[2]);
    const Dims4 n = dims4(q);
    const int64_t hkv = dims4(k).h;
    require_shape(k, {n.b, hkv, n.s, n.d}, "shape of k");
    require(v.sizes() == k.sizes(), "k and v have one shape");
    const at::ScalarType kt = k.scalar_type();
    require(v.scalar_type() == kt && (kt == at::kChar || kt == at::kBFloat16), "k and v are bf16 or int8");
    const float *ks = nullptr, *vs = nullptr;
    if (kt == at::kChar) {
        require_shape(tensor(a[5]), {n.b, hkv, n.s}, "shape of k_scale");
        require_shape(tensor(a[6]), {n.b, hkv, n.s}, "shape of v_scale");
    }
    const at::Tensor out = prefill_out(a[7], a[8], n, q);
    require_shape(out, {n.b, n.h, n.s, n.d}, "shape of out");
    void *const qp = bf16_ptr(q), *const kp = ptr(k), *const vp = ptr(v);
    if (given(a[5])) ks = f32_ptr(tensor(a[5]));
    if (given(a[6])) vs = f32_ptr(tensor(a[6]));
    void* const op = ptr(out);
    const int od = out_code(out), kd = kt == at::kChar ? SLIM_I8 : SLIM_BF16, causal = as_flag(a[4]);
    const float scale = as_float(a[3]);
    call([&](void* stream) {
        return slim_attn_prefill(qp, kp, vp, ks, vs, op, c_int(n.b), c_int(n.h), c_int(hkv), c_int(n.s), c_int(n.d), causal, scale, kd, od, stream);
    });
    return give(a[7], out);
}

void require_bf16_kv(const at::Tensor& k, const at::Tensor& v, const Dims4& n, int64_t hkv) {
    require_shape(k, {n.b, hkv, n.s, n.d}, "shape of k");
    require(v.sizes() == k.sizes(), "k and v have one shape");
    require(k.scalar_type() == at::kBFloat16 && v.scalar_type() == at::kBFloat16, "k and v are bf16");
}

// q, k, v, softmax_scale, causal, out, out_dtype
PyObject* prefill_emit(Args a) {
    const at::Tensor &q = tensor(a[0]), &k = tensor(a[1]), &v = tensor(a[2]);
    const Dims4 n = dims4(q);
    const int64_t hkv = dims4(k).h;
    require_bf16_kv(k, v, n, hkv);
    const at::Tensor out = prefill_out(a[5], a[6], n, q);
    const at::Tensor kc = make({n.b, hkv, n.s, n.d}, at::kChar, q), ks = make({n.b, hkv, n.s}, at::kFloat, q);
    const at::Tensor vc = make({n.b, hkv, n.s, n.d}, at::kChar, q), vs = make({n.b, hkv, n.s}, at::kFloat, q);
    void *const qp = bf16_ptr(q), *const kp = bf16_ptr(k), *const vp = bf16_ptr(v), *const op = ptr(out);
    int8_t *const kcp = i8_ptr(kc), *const vcp = i8_ptr(vc);
    float *const ksp = f32_ptr(ks), *const vsp = f32_ptr(vs);
    const int od = out_code(out), causal = as_flag(a[4]);
    const float scale = as_float(a[3]);
    call([&](void* stream) {
        return slim_attn_prefill_emit_int8(qp, kp, vp, op, kcp, ksp, vcp, vsp, c_int(n.b), c_int(n.h), c_int(hkv), c_int(n.s), c_int(n.d), causal, scale, od, stream);
    });
    PyObject* items[5] = {give(a[5], out), wrap(kc), wrap(ks), wrap(vc), wrap(vs)};
    return tuple_of(items);
}

// q, k, v, softmax_scale, causal, out, out_dtype, workspace
PyObject* prefill_two_sweep(Args a) {
    const at::Tensor &q = tensor(a[0]), &k = tensor(a[1]), &v = tensor(a[2]);
    const Dims4 n = dims4(q);
    const int64_t hkv = dims4(k).h;
    require_bf16_kv(k, v, n, hkv);
    const at::Tensor out = prefill_out(a[5], a[6], n, q);
    const size_t need = slim_attn_prefill_two_sweep_workspace_bytes(c_int(n.b), c_int(n.h), c_int(hkv), c_int(n.s), c_int(n.d));
    const at::Tensor ws = out_or_new(a[7], {(int64_t)std::max<size_t>(need, 16)}, at::kByte, q);
    void *const qp = bf16_ptr(q), *const kp = bf16_ptr(k), *const vp = bf16_ptr(v), *const op = ptr(out), *const wp = ptr(ws);
    const size_t ws_bytes = ws.nbytes();
    const int od = out_code(out), causal = as_flag(a[4]);
    const float scale = as_float(a[3]);
    call([&](void* stream) {
        return slim_attn_prefill_two_sweep(qp, kp, vp, op, wp, ws_bytes, c_int(n.b), c_int(n.h), c_int(hkv), c_int(n.s), c_int(n.d), causal, scale, od, stream);
    });
    return give(a[5], out);
}

// q, k, v, softmax_scale, causal, out, out_dtype
PyObject* prefill_strip(Args a) {
    const at::Tensor &q = tensor(a[0]), &k = tensor(a[1]), &v = tensor(a[2]);
    const Dims4 n = dims4(q);
    const int64_t hkv = dims4(k).h;
    require_bf16_kv(k, v, n, hkv);
    const at::Tensor out = prefill_out(a[5], a[6], n, q);
    void *const qp = bf16_ptr(q), *const kp = bf16_ptr(k), *const vp = bf16_ptr(v), *const op = ptr(out);
    const int od = out_code(out), causal = as_flag(a[4]);
    const float scale = as_float(a[3]);
    call([&](void* stream) {
        return slim_attn_prefill_strip(qp, kp, vp, op, c_int(n.b), c_int(n.h), c_int(hkv), c_int(n.s), c_int(n.d), causal, scale, od, stream);
    });
    return give(a[5], out);
}

// What the three decode calls share: q, k_codes, k_scale, v_codes, v_scale in a[0..4]
struct DecodeIn {
    int64_t b, hq, hkv, t, d;
    void* q;
    const int8_t *kc, *vc;
    const float *ks, *vs;
    explicit DecodeIn(Args a) {   // the sizes
        const at::Tensor &qt = tensor(a[0]), &kct = tensor(a[1]), &kst = tensor(a[2]), &vct = tensor(a[3]), &vst = tensor(a[4]);
        const Dims4 n = dims4(qt), c = dims4(kct);
        require(n.s == 1, "one query token per sequence");
        b = n.b, hq = n.h, hkv = c.h, t = c.s, d = n.d;
        require_shape(kct, {b, hkv, t, d}, "shape of k_codes");
        require(vct.sizes() == kct.sizes(), "k_codes and v_codes have one shape");
        require_shape(kst, {b, hkv, t}, "shape of k_scale");
        require_shape(vst, {b, hkv, t}, "shape of v_scale");
    }
    void take_pointers(Args a) {   // (once the results are allocated: that may let other threads run)
        const at::Tensor &qt = tensor(a[0]), &kct = tensor(a[1]), &kst = tensor(a[2]), &vct = tensor(a[3]), &vst = tensor(a[4]);
        q = bf16_ptr(qt), kc = i8_ptr(kct), ks = f32_ptr(kst), vc = i8_ptr(vct), vs = f32_ptr(vst);
    }
};

// q, k_codes, k_scale, v_codes, v_scale, softmax_scale, causal, out, workspace, and kv_lens with VARLEN
template <bool VARLEN>
PyObject* decode(Args a) {
    DecodeIn in(a);
    const at::Tensor& q = tensor(a[0]);
    if (VARLEN) require_shape(tensor(a[9]), {in.b}, "one length per sequence");
    const at::Tensor out = out_or_new(a[7], {in.b, in.hq, 1, in.d}, at::kBFloat16, q);
    require_room(out, in.b * in.hq * in.d, "out is too small");
    at::Tensor fresh_ws;
    if (!given(a[8])) {
        const size_t need = slim_attn_decode_int8_workspace_bytes(c_int(in.b), c_int(in.hq), c_int(in.hkv), c_int(in.t), c_int(in.d));
        fresh_ws = make({(int64_t)std::max<size_t>(need, 16)}, at::kByte, q);
    }
    const at::Tensor& ws = given(a[8]) ? tensor(a[8]) : fresh_ws;
    in.take_pointers(a);
    const int32_t* const lens = VARLEN ? i32_ptr(tensor(a[9])) : nullptr;
    void *const op = bf16_ptr(out), *const wp = ptr(ws);
    const size_t ws_bytes = ws.nbytes();
    const int causal = as_flag(a[6]);
    const float scale = as_float(a[5]);
    call([&](void* stream) {
        return !VARLEN ? slim_attn_decode_int8(in.q, in.kc, in.ks, in.vc, in.vs, op, wp, ws_bytes, c_int(in.b), c_int(in.hq),
                                                       c_int(in.hkv), c_int(in.t), c_int(in.d), causal, scale, stream)
                               : slim_attn_decode_int8_varlen(in.q, in.kc, in.ks, in.vc, in.vs, lens, op, wp, ws_bytes, c_int(in.b),
                                                              c_int(in.hq), c_int(in.hkv), c_int(in.t), c_int(in.d), causal, scale, stream);
    });
    return give(a[7], out);
}

// q, k_codes, k_scale, v_codes, v_scale, softmax_scale, out, causal
PyObject* decode_static(Args a) {
    DecodeIn in(a);
    const at::Tensor& out = tensor(a[6]);
    require_shape(out, {in.b, in.hq, 1, in.d}, "shape of out");
    in.take_pointers(a);
    void* const op = bf16_ptr(out);
    const int causal = as_flag(a[7]);
    const float scale = as_float(a[5]);
    call([&](void* stream) {
        return slim_attn_decode_int8_static(in.q, in.kc, in.ks, in.vc, in.vs, op, c_int(in.b), c_int(in.hq), c_int(in.hkv), c_int(in.t),
                                            c_int(in.d), causal, scale, stream);
    });
    return give(a[6], out);
}

template <PyObject* (*F)(Args), int N>
PyObject* entry(PyObject*, PyObject* const* args, Py_ssize_t n) {
    if (n != N) {
        PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
        return nullptr;
    }
    HANDLE_TH_ERRORS
    try {
        return F(args);
    } catch (const Failed&) {
        return nullptr;
    }
    END_HANDLE_TH_ERRORS
}

PyObject* set_raise_status(PyObject*, PyObject* f) {
    Py_INCREF(f);
    Py_XSETREF(g_raise_status, f);
    Py_RETURN_NONE;
}

#define SLIM_ENTRY(name, fn, n) {name, (PyCFunction)(void (*)(void))(&entry<fn, n>), METH_FASTCALL, nullptr}
PyMethodDef g_methods[] = {
    SLIM_ENTRY("kv_quant", kv_quant, 3),
    SLIM_ENTRY("kv_quant_pair", kv_quant_pair, 6),
    SLIM_ENTRY("kv_quant_append", kv_quant_append, 4),
    SLIM_ENTRY("prefill", prefill, 9),
    SLIM_ENTRY("prefill_emit", prefill_emit, 7),
    SLIM_ENTRY("prefill_two_sweep", prefill_two_sweep, 8),
    SLIM_ENTRY("prefill_strip", prefill_strip, 7),
    SLIM_ENTRY("decode", decode<false>, 9),
    SLIM_ENTRY("decode_varlen", decode<true>, 10),
    SLIM_ENTRY("decode_static", decode_static, 8),
    {"set_raise_status", set_raise_status, METH_O, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_slimbind", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__slimbind() { return PyModule_Create(&g_module); }
