// Python side of the C ABI (include/rcp.h): argument checks and marshalling from torch tensors.
//
// A decode step is a chain of launches of 2 to 7 us each, issued by one host thread, so what a call costs the
// host bounds the step as soon as it exceeds the kernel: 8 us a call when tensors were taken apart and checked
// in Python and handed over through ctypes, against 1 us of work of its own here.  Each function takes its
// arguments by position (the keyword arguments and defaults live in the package's __init__.py), reads the tensor
// objects directly, takes the current stream of the current device and calls the library with the interpreter
// lock released.  ValueError: a tensor that does not fit its use; RcpError: the library's own status.
#include <Python.h>

#include <ATen/ops/empty.h>
#include <c10/core/DefaultDtype.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/autograd/python_variable.h>

#include <climits>
#include <cstdint>
#include <string>
#include <vector>

#include "rcp.h"

namespace {

using at::Tensor;
using Args = PyObject* const*;

PyObject* g_error = nullptr;  // RcpError(code, message)

struct Bad {  // -> ValueError
    std::string what;
};
struct Raised {};  // a Python error is already set
struct Status {  // -> RcpError
    int rc;
};

inline void require(bool ok, const char* message)
{
    if (__builtin_expect(!ok, 0)) throw Bad{message};
}

inline const Tensor& tensor(PyObject* o, const char* what)
{
    if (__builtin_expect(!THPVariable_Check(o), 0)) throw Bad{std::string(what) + " must be a contiguous CUDA tensor"};
    return THPVariable_Unpack(o);
}

inline void* dev(const Tensor& t, const char* what)
{
    if (__builtin_expect(!t.is_cuda() || !t.is_contiguous(), 0)) throw Bad{std::string(what) + " must be a contiguous CUDA tensor"};
    return t.data_ptr();
}

inline void* dev(PyObject* o, const char* what) { return dev(tensor(o, what), what); }

inline bool none(PyObject* o) { return o == Py_None; }

inline void* opt(PyObject* o, const char* what) { return none(o) ? nullptr : dev(o, what); }

// The library counts in 32 bits: what does not fit is refused here, before a check could pass on its low half.
inline int narrow(int64_t v)
{
    require(v >= INT_MIN && v <= INT_MAX, "sizes, counts and positions must fit a 32-bit integer");
    return static_cast<int>(v);
}

inline int integer(PyObject* o)
{
    int overflow = 0;
    const long long v = PyLong_AsLongLongAndOverflow(o, &overflow);
    if (v == -1 && overflow == 0 && PyErr_Occurred()) throw Raised{};
    return narrow(overflow != 0 ? INT64_MAX : v);
}

// A position or length: anything that int() takes.
inline int position(PyObject* o)
{
    if (__builtin_expect(PyLong_Check(o), 1)) return integer(o);
    PyObject* const whole = PyNumber_Long(o);
    if (whole == nullptr) throw Raised{};
    int overflow = 0;
    const long long v = PyLong_AsLongLongAndOverflow(whole, &overflow);
    Py_DECREF(whole);
    return narrow(overflow != 0 ? INT64_MAX : v);
}

inline float real(PyObject* o)
{
    const double v = PyFloat_AsDouble(o);
    if (v == -1.0 && PyErr_Occurred()) throw Raised{};
    return static_cast<float>(v);
}

inline bool truth(PyObject* o)
{
    const int v = PyObject_IsTrue(o);
    if (v < 0) throw Raised{};
    return v != 0;
}

inline const rcp_rotation* rotation(PyObject* o)  // address of the descriptor, 0 = none
{
    void* p = PyLong_AsVoidPtr(o);
    if (p == nullptr && PyErr_Occurred()) throw Raised{};
    return static_cast<const rcp_rotation*>(p);
}

inline int dtype_code(const Tensor& t)
{
    switch (t.scalar_type()) {
        case at::kHalf: return RCP_F16;
        case at::kFloat: return RCP_F32;
        case at::kBFloat16: return RCP_BF16;
        default: return -1;
    }
}

inline rcp_dtype in_dtype(const Tensor& t, const char* message)
{
    const int d = dtype_code(t);
    require(d >= 0, message);
    return static_cast<rcp_dtype>(d);
}

inline rcp_dtype out_code(const Tensor& t, const char* message)
{
    const at::ScalarType s = t.scalar_type();
    require(s == at::kHalf || s == at::kFloat, message);
    return s == at::kHalf ? RCP_F16 : RCP_F32;
}

inline int64_t nbytes(const Tensor& t) { return static_cast<int64_t>(t.nbytes()); }

inline at::ScalarType scalar_type(PyObject* o)
{
    if (none(o)) return c10::get_default_dtype_as_scalartype();  // as torch.empty has it
    if (!THPDtype_Check(o)) throw Bad{"out_dtype must be a torch.dtype"};
    return reinterpret_cast<THPDtype*>(o)->scalar_type;
}

inline Tensor empty_like_device(at::IntArrayRef shape, at::ScalarType type, const Tensor& where)
{
    return at::empty(shape, at::TensorOptions().dtype(type).device(where.device()));
}

// An argument that the caller may leave out: the object itself, or a new tensor.
struct Result {
    Tensor t;
    PyObject* o = nullptr;  // borrowed; null when the tensor was made here
    PyObject* give() const
    {
        if (o == nullptr) return THPVariable_Wrap(t);
        Py_INCREF(o);
        return o;
    }
};

inline Result given(PyObject* o, const char* what)
{
    Result r;
    r.t = tensor(o, what);
    r.o = o;
    return r;
}

inline Result output(PyObject* o, PyObject* dtype, at::IntArrayRef shape, const Tensor& where)
{
    if (!none(o)) return given(o, "out");
    Result r;
    r.t = empty_like_device(shape, scalar_type(dtype), where);
    return r;
}

// int32 partial sums: given, wanted, or neither
inline Result sums(PyObject* o, PyObject* want, at::IntArrayRef shape, const Tensor& where)
{
    if (!none(o)) return given(o, "partial_sums");
    Result r;
    if (truth(want)) r.t = empty_like_device(shape, at::kInt, where);
    return r;
}

inline int32_t* sums_ptr(const Result& r, int64_t count, const char* message)
{
    if (!r.t.defined()) return nullptr;
    require(r.t.scalar_type() == at::kInt && r.t.numel() >= count, message);
    return static_cast<int32_t*>(dev(r.t, "partial_sums"));
}

inline PyObject* pair(PyObject* a, PyObject* b)
{
    if (a == nullptr || b == nullptr) {
        Py_XDECREF(a);
        Py_XDECREF(b);
        throw Raised{};
    }
    PyObject* t = PyTuple_New(2);
    if (t == nullptr) throw Raised{};
    PyTuple_SET_ITEM(t, 0, a);
    PyTuple_SET_ITEM(t, 1, b);
    return t;
}

inline PyObject* result(const Result& out, const Result& P) { return P.t.defined() ? pair(out.give(), P.give()) : out.give(); }

inline PyObject* nothing()
{
    Py_INCREF(Py_None);
    return Py_None;
}

template <class F>
inline void call(F f)  // f(stream) -> status, without the interpreter lock (a full queue makes a launch wait)
{
    void* const stream = c10::hip::getCurrentHIPStream().stream();
    PyThreadState* const saved = PyEval_SaveThread();
    const int rc = f(stream);
    PyEval_RestoreThread(saved);
    if (__builtin_expect(rc != RCP_OK, 0)) throw Status{rc};
}

// ---- linear layers ----------------------------------------------------------------------------------
struct Weights {
    const void *packed, *codebook;
    int N, K;
};

// packed, codebook, N, K at a[0..3]; `weight_eighths` bits of index storage per weight in units of 1/8 byte
inline Weights weights(Args a, int weight_eighths, int64_t levels_per_row_unit, int64_t units, const char* message)
{
    const Tensor &p = tensor(a[0], "packed"), &c = tensor(a[1], "codebook");
    Weights w;
    w.N = integer(a[2]);
    w.K = integer(a[3]);
    const int64_t need = static_cast<int64_t>(weight_eighths) * w.N * w.K / 8;
    require(nbytes(p) >= need && c.numel() >= levels_per_row_unit * w.N * units, message);
    w.packed = dev(p, "packed");
    w.codebook = dev(c, "codebook");
    return w;
}

constexpr const char* kNK = "packed / codebook buffers do not match N, K";
constexpr const char* kNKG = "packed / codebook buffers do not match N, K, group";
constexpr const char* kX = "x must hold K values of float16, bfloat16 or float32";
constexpr const char* kXType = "x must be float16, bfloat16 or float32";
constexpr const char* kOutN = "out must be float16 or float32 with N elements";
constexpr const char* kP2 = "partial_sums must be int32 [1, N, 4]";
constexpr const char* kPG = "partial_sums must be int32 [N, K/group, 4]";

inline int groups_of(int K, int group)
{
    if (group == 0) {
        PyErr_SetString(PyExc_ZeroDivisionError, "integer division or modulo by zero");
        throw Raised{};
    }
    const int g = K / group;
    return g > 1 ? g : 1;
}

// packed, codebook, N, K, xq, scale, M, out, out_dtype, partial_sums, want
PyObject* w2a4_gemv(Args a)
{
    const int N = integer(a[2]), K = integer(a[3]), M = integer(a[6]);
    const Tensor& where = tensor(a[0], "packed");
    const Result out = output(a[7], a[8], {M, N}, where);
    const rcp_dtype od = out_code(out.t, "out must be float16 or float32");
    const Result P = sums(a[9], a[10], {M, N, 4}, where);
    const Weights w = weights(a, 2, 4, 1, kNK);
    const Tensor &xq = tensor(a[4], "xq"), &scale = tensor(a[5], "scale");
    const int64_t mn = static_cast<int64_t>(M) * N;
    require(nbytes(xq) >= static_cast<int64_t>(M) * K / 2 && scale.numel() >= M && out.t.numel() >= mn,
            "xq / scale / out buffers do not match M, N, K");
    int32_t* const p = sums_ptr(P, 4 * mn, "partial_sums must be int32 [M, N, 4]");
    void *const x = dev(xq, "xq"), *const s = dev(scale, "scale"), *const o = dev(out.t, "out");
    call([&](void* st) { return rcp_w2a4_gemv(w.packed, w.codebook, N, K, x, s, M, o, od, p, st); });
    return result(out, P);
}

// packed, codebook, N, K, x, rotation, clip_ratio, out, out_dtype, xq_out, scale_out, partial_sums, want
PyObject* rotate_quant_w2a4_gemv(Args a)
{
    const int N = integer(a[2]), K = integer(a[3]);
    const Tensor &x = tensor(a[4], "x"), &where = tensor(a[0], "packed");
    require(x.numel() == K, kX);
    const rcp_dtype xd = in_dtype(x, kX);
    const rcp_rotation* const rot = rotation(a[5]);
    const float ratio = real(a[6]);
    const Result out = output(a[7], a[8], {1, N}, where);
    const rcp_dtype od = out_code(out.t, kOutN);
    require(out.t.numel() >= N, kOutN);
    const Result P = sums(a[11], a[12], {1, N, 4}, where);
    const Weights w = weights(a, 2, 4, 1, kNK);
    if (!none(a[9])) require(nbytes(tensor(a[9], "xq_out")) >= K / 2, "xq_out too small");
    int32_t* const p = sums_ptr(P, 4 * static_cast<int64_t>(N), kP2);
    void *const xp = dev(x, "x"), *const o = dev(out.t, "out"), *const xo = opt(a[9], "xq_out"), *const so = opt(a[10], "scale_out");
    call([&](void* st) { return rcp_rotate_quant_w2a4_gemv(w.packed, w.codebook, N, K, xp, xd, rot, ratio, o, od, xo, so, p, st); });
    return result(out, P);
}

// packed, codebook, N, K, x, clip_ratio, group, out, out_dtype, xq_out, scale_out, partial_sums, want
PyObject* quant_w2a4_gemv_grouped(Args a)
{
    const int N = integer(a[2]), K = integer(a[3]), group = integer(a[6]), NG = groups_of(K, group);
    const Tensor &x = tensor(a[4], "x"), &where = tensor(a[0], "packed");
    require(x.numel() == K, kX);
    const rcp_dtype xd = in_dtype(x, kX);
    const float ratio = real(a[5]);
    const Result out = output(a[7], a[8], {1, N}, where);
    const rcp_dtype od = out_code(out.t, kOutN);
    require(out.t.numel() >= N, kOutN);
    const Result P = sums(a[11], a[12], {N, NG, 4}, where);
    const Weights w = weights(a, 2, 4, NG, kNKG);
    if (!none(a[9])) require(nbytes(tensor(a[9], "xq_out")) >= K / 2, "xq_out too small");
    int32_t* const p = sums_ptr(P, 4 * static_cast<int64_t>(N) * NG, kPG);
    void *const xp = dev(x, "x"), *const o = dev(out.t, "out"), *const xo = opt(a[9], "xq_out"), *const so = opt(a[10], "scale_out");
    call([&](void* st) { return rcp_quant_w2a4_gemv_grouped(w.packed, w.codebook, N, K, group, xp, xd, ratio, o, od, xo, so, p, st); });
    return result(out, P);
}

// packed, codebook, N, K, xq, scale, group, out, out_dtype, partial_sums, want
PyObject* w2a4_gemv_grouped(Args a)
{
    const int N = integer(a[2]), K = integer(a[3]), group = integer(a[6]), NG = groups_of(K, group);
    const Tensor& where = tensor(a[0], "packed");
    const Result out = output(a[7], a[8], {1, N}, where);
    const rcp_dtype od = out_code(out.t, kOutN);
    require(out.t.numel() >= N, kOutN);
    const Result P = sums(a[9], a[10], {N, NG, 4}, where);
    const Weights w = weights(a, 2, 4, NG, kNKG);
    const Tensor &xq = tensor(a[4], "xq"), &scale = tensor(a[5], "scale");
    require(nbytes(xq) >= K / 2 && scale.numel() >= 1, "xq / scale buffers do not match K");
    int32_t* const p = sums_ptr(P, 4 * static_cast<int64_t>(N) * NG, kPG);
    void *const x = dev(xq, "xq"), *const s = dev(scale, "scale"), *const o = dev(out.t, "out");
    call([&](void* st) { return rcp_w2a4_gemv_grouped(w.packed, w.codebook, N, K, group, x, s, o, od, p, st); });
    return result(out, P);
}

// packed, codebook, N, K, xq, scale, M, group, out, out_dtype, partial_sums, want
PyObject* w2a4_gemm_grouped(Args a)
{
    const int N = integer(a[2]), K = integer(a[3]), M = integer(a[6]), group = integer(a[7]), NG = groups_of(K, group);
    const Tensor& where = tensor(a[0], "packed");
    const int64_t mn = static_cast<int64_t>(M) * N;
    const Result out = output(a[8], a[9], {M, N}, where);
    const rcp_dtype od = out_code(out.t, "out must be float16 or float32 with M*N elements");
    require(out.t.numel() >= mn, "out must be float16 or float32 with M*N elements");
    const Result P = sums(a[10], a[11], {M, N, NG, 4}, where);
    const Weights w = weights(a, 2, 4, NG, kNKG);
    const Tensor &xq = tensor(a[4], "xq"), &scale = tensor(a[5], "scale");
    require(nbytes(xq) >= static_cast<int64_t>(M) * K / 2 && scale.numel() >= M, "xq / scale buffers do not match M, K");
    int32_t* const p = sums_ptr(P, 4 * mn * NG, "partial_sums must be int32 [M, N, K/group, 4]");
    void *const x = dev(xq, "xq"), *const s = dev(scale, "scale"), *const o = dev(out.t, "out");
    call([&](void* st) { return rcp_w2a4_gemm_grouped(w.packed, w.codebook, N, K, group, x, s, M, o, od, p, st); });
    return result(out, P);
}

// packed, codebook, N, K, x, out, out_dtype
PyObject* w2a16_gemv(Args a)
{
    const int N = integer(a[2]), K = integer(a[3]);
    const Tensor& x = tensor(a[4], "x");
    require(x.numel() == K, kX);
    const rcp_dtype xd = in_dtype(x, kX);
    const Result out = output(a[5], a[6], {1, N}, tensor(a[0], "packed"));
    const rcp_dtype od = out_code(out.t, kOutN);
    require(out.t.numel() >= N, kOutN);
    const Weights w = weights(a, 2, 4, 1, kNK);
    void *const xp = dev(x, "x"), *const o = dev(out.t, "out");
    call([&](void* st) { return rcp_w2a16_gemv(w.packed, w.codebook, N, K, xp, xd, o, od, st); });
    return out.give();
}

// packed, codebook, N, K, xq, scale, out, out_dtype, partial_sums, want
PyObject* w3a4_gemv(Args a)
{
    const int N = integer(a[2]), K = integer(a[3]);
    const Tensor& where = tensor(a[0], "packed");
    const Result out = output(a[6], a[7], {1, N}, where);
    const rcp_dtype od = out_code(out.t, kOutN);
    require(out.t.numel() >= N, kOutN);
    const Result P = sums(a[8], a[9], {N, 8}, where);
    const Weights w = weights(a, 3, 8, 1, kNK);
    const Tensor &xq = tensor(a[4], "xq"), &scale = tensor(a[5], "scale");
    require(nbytes(xq) >= K / 2 && scale.numel() >= 1, "xq / scale buffers do not match K");
    int32_t* const p = sums_ptr(P, 8 * static_cast<int64_t>(N), "partial_sums must be int32 [N, 8]");
    void *const x = dev(xq, "xq"), *const s = dev(scale, "scale"), *const o = dev(out.t, "out");
    call([&](void* st) { return rcp_w3a4_gemv(w.packed, w.codebook, N, K, x, s, o, od, p, st); });
    return result(out, P);
}

// packed, codebook, N, K, x, clip_ratio, out, out_dtype, xq_out, scale_out, partial_sums, want
PyObject* quant_w3a4_gemv(Args a)
{
    const int N = integer(a[2]), K = integer(a[3]);
    const Tensor &x = tensor(a[4], "x"), &where = tensor(a[0], "packed");
    require(x.numel() == K, kX);
    const rcp_dtype xd = in_dtype(x, kX);
    const float ratio = real(a[5]);
    const Result out = output(a[6], a[7], {1, N}, where);
    const rcp_dtype od = out_code(out.t, kOutN);
    require(out.t.numel() >= N, kOutN);
    const Result P = sums(a[10], a[11], {N, 8}, where);
    const Weights w = weights(a, 3, 8, 1, kNK);
    if (!none(a[8])) require(nbytes(tensor(a[8], "xq_out")) >= K / 2, "xq_out too small");
    int32_t* const p = sums_ptr(P, 8 * static_cast<int64_t>(N), "partial_sums must be int32 [N, 8]");
    void *const xp = dev(x, "x"), *const o = dev(out.t, "out"), *const xo = opt(a[8], "xq_out"), *const so = opt(a[9], "scale_out");
    call([&](void* st) { return rcp_quant_w3a4_gemv(w.packed, w.codebook, N, K, xp, xd, ratio, o, od, xo, so, p, st); });
    return result(out, P);
}

// ---- activations --------------------------------------------------------------------------------------
// x of shape [M, K], or [K] for one token
inline void rows_of(const Tensor& x, int& M, int& K)
{
    require(x.dim() == 1 || x.dim() == 2, "x must be [M, K] or [K]");
    M = x.dim() == 1 ? 1 : narrow(x.size(0));
    K = narrow(x.size(-1));
}

// x, rotation, clip_ratio, xq_out, scale_out, workspace
PyObject* rotate_quant_act(Args a)
{
    const Tensor& x = tensor(a[0], "x");
    int M, K;
    rows_of(x, M, K);
    const rcp_dtype xd = in_dtype(x, kXType);
    const rcp_rotation* const rot = rotation(a[1]);
    const float ratio = real(a[2]);
    Result xq, scale;
    if (none(a[3])) xq.t = empty_like_device({M, K / 2 > 1 ? K / 2 : 1}, at::kByte, x);
    else xq = given(a[3], "xq_out");
    if (none(a[4])) scale.t = empty_like_device({M}, at::kHalf, x);
    else scale = given(a[4], "scale_out");
    Tensor work;
    if (!none(a[5])) work = tensor(a[5], "workspace");
    else if (const size_t need = rcp_act_workspace_bytes(M, K, rot))
        work = empty_like_device({static_cast<int64_t>(need)}, at::kByte, x);
    void* const ws = work.defined() ? dev(work, "workspace") : nullptr;
    const size_t ws_bytes = work.defined() ? work.nbytes() : 0;
    void *const xp = dev(x, "x"), *const xo = dev(xq.t, "xq_out"), *const so = dev(scale.t, "scale_out");
    call([&](void* st) { return rcp_rotate_quant_act(xp, xd, M, K, rot, ratio, xo, so, ws, ws_bytes, st); });
    return pair(xq.give(), scale.give());
}

// x, rotation, clip_ratio, xq_out, scale_out
PyObject* rotate_quant_act_static(Args a)
{
    const Tensor& x = tensor(a[0], "x");
    int M, K;
    rows_of(x, M, K);
    const rcp_dtype xd = in_dtype(x, kXType);
    const rcp_rotation* const rot = rotation(a[1]);
    const float ratio = real(a[2]);
    const Result xq = given(a[3], "xq_out"), scale = given(a[4], "scale_out");
    void *const xp = dev(x, "x"), *const xo = dev(xq.t, "xq_out"), *const so = dev(scale.t, "scale_out");
    call([&](void* st) { return rcp_rotate_quant_act_static(xp, xd, M, K, rot, ratio, xo, so, st); });
    return pair(xq.give(), scale.give());
}

// x, rotation, y_out
PyObject* rotate_act(Args a)
{
    const Tensor& x = tensor(a[0], "x");
    int M, K;
    rows_of(x, M, K);
    const rcp_dtype xd = in_dtype(x, kXType);
    const rcp_rotation* const rot = rotation(a[1]);
    Result y;
    if (none(a[2])) y.t = empty_like_device({M, K}, at::kFloat, x);
    else y = given(a[2], "y_out");
    require(y.t.scalar_type() == at::kFloat && y.t.numel() >= static_cast<int64_t>(M) * K, "y_out must be float32 [M, K]");
    void *const xp = dev(x, "x"), *const yp = dev(y.t, "y_out");
    call([&](void* st) { return rcp_rotate_act(xp, xd, M, K, rot, static_cast<float*>(yp), st); });
    return y.give();
}

// ---- export -------------------------------------------------------------------------------------------
inline const float* learnt(PyObject* o, const char* name)
{
    const Tensor& t = tensor(o, name);
    if (t.scalar_type() != at::kFloat) throw Bad{std::string(name) + " must be float32"};
    return static_cast<const float*>(dev(t, name));
}

inline void matrix_of(const Tensor& W, int& N, int& K, rcp_dtype& dt)
{
    require(W.dim() == 2, "W must be [N, K]");
    N = narrow(W.size(0));
    K = narrow(W.size(1));
    dt = in_dtype(W, "W must be float16, bfloat16 or float32");
}

inline int64_t count(PyObject* o) { return THPVariable_Unpack(o).numel(); }

// W, clip_lo, clip_hi, part, packed_out, codebook_out
PyObject* pack_weights(Args a)
{
    const Tensor& W = tensor(a[0], "W");
    int N, K;
    rcp_dtype wd;
    matrix_of(W, N, K, wd);
    const float *const lo = learnt(a[1], "clip_lo"), *const hi = learnt(a[2], "clip_hi"), *const part = learnt(a[3], "part");
    require(count(a[1]) == N && count(a[2]) == N && count(a[3]) == 3 * static_cast<int64_t>(N), "clip_lo / clip_hi / part do not match N");
    Result p, c;
    const int64_t need = static_cast<int64_t>(rcp_packed_bytes(N, K));
    if (none(a[4])) p.t = empty_like_device({need > 1 ? need : 1}, at::kByte, W);
    else p = given(a[4], "packed_out");
    if (none(a[5])) c.t = empty_like_device({N, 4}, at::kHalf, W);
    else c = given(a[5], "codebook_out");
    void *const w = dev(W, "W"), *const po = dev(p.t, "packed_out"), *const co = dev(c.t, "codebook_out");
    call([&](void* st) { return rcp_pack_weights(w, wd, N, K, lo, hi, part, po, co, st); });
    return pair(p.give(), c.give());
}

// W, clip_lo, clip_hi, part, group, packed_out, codebook_out
PyObject* pack_weights_grouped(Args a)
{
    const Tensor& W = tensor(a[0], "W");
    int N, K;
    rcp_dtype wd;
    matrix_of(W, N, K, wd);
    const int group = integer(a[4]);
    groups_of(K, group);  // group = 0 is an error
    const int NG = K / group;
    const int64_t units = static_cast<int64_t>(N) * NG;
    const float *const lo = learnt(a[1], "clip_lo"), *const hi = learnt(a[2], "clip_hi"), *const part = learnt(a[3], "part");
    require(count(a[1]) == units && count(a[2]) == units && count(a[3]) == 3 * units, "clip_lo / clip_hi / part do not match N, K/group");
    Result p, c;
    const int64_t need = static_cast<int64_t>(N) * K / 4;
    if (none(a[5])) p.t = empty_like_device({need > 1 ? need : 1}, at::kByte, W);
    else p = given(a[5], "packed_out");
    if (none(a[6])) c.t = empty_like_device({N / 4 > 1 ? N / 4 : 1, NG > 1 ? NG : 1, 4, 4}, at::kHalf, W);
    else c = given(a[6], "codebook_out");
    require(nbytes(p.t) >= need && c.t.numel() >= 4 * units, "packed_out / codebook_out too small");
    void *const w = dev(W, "W"), *const po = dev(p.t, "packed_out"), *const co = dev(c.t, "codebook_out");
    call([&](void* st) { return rcp_pack_weights_grouped(w, wd, N, K, group, lo, hi, part, po, co, st); });
    return pair(p.give(), c.give());
}

// W, clip_lo, clip_hi, frac, grid (eight floats), packed_out, codebook_out
PyObject* pack_weights_w3(Args a)
{
    const Tensor& W = tensor(a[0], "W");
    int N, K;
    rcp_dtype wd;
    matrix_of(W, N, K, wd);
    const float* learn[3];
    const char* const names[3] = {"clip_lo", "clip_hi", "frac"};
    for (int i = 0; i < 3; ++i) {
        const Tensor& t = tensor(a[1 + i], names[i]);
        if (t.scalar_type() != at::kFloat || t.numel() != N) throw Bad{std::string(names[i]) + " must be float32 with N elements"};
        learn[i] = static_cast<const float*>(dev(t, names[i]));
    }
    float grid[8];
    {
        PyObject* s = PySequence_Fast(a[4], "grid must be a sequence");
        if (s == nullptr) throw Raised{};
        const bool eight = PySequence_Fast_GET_SIZE(s) == 8;
        if (eight)
            for (int i = 0; i < 8; ++i) grid[i] = static_cast<float>(PyFloat_AsDouble(PySequence_Fast_GET_ITEM(s, i)));
        Py_DECREF(s);
        if (PyErr_Occurred()) throw Raised{};
        require(eight, "grid must hold eight values");
    }
    Result p, c;
    const int64_t need = 3 * static_cast<int64_t>(N) * K / 8;
    if (none(a[5])) p.t = empty_like_device({need > 1 ? need : 1}, at::kByte, W);
    else p = given(a[5], "packed_out");
    if (none(a[6])) c.t = empty_like_device({N, 8}, at::kHalf, W);
    else c = given(a[6], "codebook_out");
    require(nbytes(p.t) >= need && c.t.numel() >= 8 * static_cast<int64_t>(N), "packed_out / codebook_out buffers do not match N, K");
    void *const w = dev(W, "W"), *const po = dev(p.t, "packed_out"), *const co = dev(c.t, "codebook_out");
    call([&](void* st) { return rcp_pack_weights_w3(w, wd, N, K, learn[0], learn[1], learn[2], grid, po, co, st); });
    return pair(p.give(), c.give());
}

// ---- 4-bit KV cache -------------------------------------------------------------------------------------
constexpr int64_t D = RCP_KV_HEAD_DIM;

struct Cache {
    void *codes, *params;
    int heads, S_max;
};

// codes uint8 [heads, S_max, 64] and params uint8 [heads, S_max, 4]; heads / S_max < 0: not known beforehand
inline Cache cache(PyObject* codes, PyObject* params, int64_t heads, int64_t S_max, const char* cname, const char* pname, const char* message)
{
    const Tensor &c = tensor(codes, cname), &p = tensor(params, pname);
    require(c.scalar_type() == at::kByte && p.scalar_type() == at::kByte && c.dim() == 3 && p.dim() == 3, message);
    if (heads < 0) heads = c.size(0);
    if (S_max < 0) S_max = c.size(1);
    require(c.size(0) == heads && c.size(1) == S_max && c.size(2) == D / 2 && p.size(0) == heads && p.size(1) == S_max &&
                p.size(2) == 4 && c.is_contiguous() && p.is_contiguous(),
            message);
    return {dev(c, cname), dev(p, pname), narrow(heads), narrow(S_max)};
}

inline void heads_of(const Tensor& x, const char* message) { require(x.dim() == 3 && x.size(2) == D && x.is_contiguous(), message); }

constexpr const char* kCodes = "codes must be uint8 [H, S_max, 64] and params uint8 [H, S_max, 4], contiguous";
constexpr const char* kCaches = "cache buffers must be uint8 [H_kv, S_max, 64] / [H_kv, S_max, 4], contiguous";
constexpr const char* kPool = "cache buffers must be uint8 [B*H_kv, S_max, 64] / [B*H_kv, S_max, 4], contiguous";

// x, pos, codes, params, clip_ratio, rotate
PyObject* kv4_append(Args a)
{
    const Tensor& x = tensor(a[0], "x");
    heads_of(x, "x must be contiguous [n_tokens, H, 128]");
    const Cache c = cache(a[2], a[3], x.size(1), -1, "codes", "params", kCodes);
    const int n = narrow(x.size(0)), H = narrow(x.size(1)), pos = position(a[1]);
    const float ratio = real(a[4]);
    const int rotate = truth(a[5]);
    if (n == 0) return nothing();  // an empty tensor has no device pointer to hand over
    const rcp_dtype xd = in_dtype(x, kXType);
    void* const xp = dev(x, "x");
    call([&](void* st) { return rcp_kv4_append(xp, xd, n, H, c.S_max, pos, rotate, ratio, c.codes, c.params, st); });
    return nothing();
}

// k, v, pos, k_codes, k_params, v_codes, v_params, clip_ratio, rotate_k
PyObject* kv4_append_kv(Args a)
{
    const Tensor &k = tensor(a[0], "k"), &v = tensor(a[1], "v");
    const char* const kv = "k and v must be contiguous [n_tokens, H, 128] of one dtype";
    heads_of(k, kv);
    require(v.sizes() == k.sizes() && v.scalar_type() == k.scalar_type() && v.is_contiguous(), kv);
    const char* const one = "codes must be uint8 [H, S_max, 64] and params uint8 [H, S_max, 4], contiguous, one S_max";
    const Cache kc = cache(a[3], a[4], k.size(1), -1, "k_codes", "k_params", one);
    const Cache vc = cache(a[5], a[6], k.size(1), kc.S_max, "v_codes", "v_params", one);
    const int n = narrow(k.size(0)), H = narrow(k.size(1)), pos = position(a[2]);
    const float ratio = real(a[7]);
    const int rotate = truth(a[8]);
    if (n == 0) return nothing();
    const rcp_dtype xd = in_dtype(k, "k and v must be float16, bfloat16 or float32");
    void *const kp = dev(k, "k"), *const vp = dev(v, "v");
    call([&](void* st) {
        return rcp_kv4_append_kv(kp, vp, xd, n, H, kc.S_max, pos, rotate, ratio, kc.codes, kc.params, vc.codes, vc.params, st);
    });
    return nothing();
}

// q, S, k_codes, k_params, v_codes, v_params, softmax_scale, out, out_dtype, workspace, rotate
PyObject* kv4_attn_decode(Args a)
{
    const Tensor& q = tensor(a[0], "q");
    require(q.dim() == 2 && q.size(1) == D && q.is_contiguous(), "q must be contiguous [H_q, 128]");
    const Cache k = cache(a[2], a[3], -1, -1, "k_codes", "k_params", kCaches);
    const Cache v = cache(a[4], a[5], k.heads, k.S_max, "v_codes", "v_params", kCaches);
    const int H_q = narrow(q.size(0)), S = position(a[1]);
    const float scale = real(a[6]);
    const Result out = output(a[7], a[8], {H_q, D}, q);
    const rcp_dtype od = out_code(out.t, "out must be float16 or float32 [H_q, 128]");
    require(out.t.numel() >= H_q * D, "out must be float16 or float32 [H_q, 128]");
    Tensor work;
    if (none(a[9])) {
        const int64_t need = static_cast<int64_t>(rcp_kv4_workspace_bytes(H_q, S));
        work = empty_like_device({need > 16 ? need : 16}, at::kByte, q);
    } else
        work = tensor(a[9], "workspace");
    const bool rotate = truth(a[10]);
    const rcp_dtype qd = in_dtype(q, "q must be float16, bfloat16 or float32");
    void *const qp = dev(q, "q"), *const o = dev(out.t, "out"), *const ws = dev(work, "workspace");
    const auto f = rotate ? rcp_kv4_rotate_attn_decode : rcp_kv4_attn_decode;
    call([&](void* st) {
        return f(qp, qd, H_q, k.heads, k.S_max, S, k.codes, k.params, v.codes, v.params, scale, o, od, ws,
                 work.nbytes(), st);
    });
    return out.give();
}

inline std::vector<int> integers(PyObject* o)
{
    if (PyObject_Size(o) < 0) throw Raised{};  // (an iterator has no length)
    PyObject* s = PySequence_Fast(o, "a sequence of integers is wanted");
    if (s == nullptr) throw Raised{};
    const Py_ssize_t n = PySequence_Fast_GET_SIZE(s);
    std::vector<int> r(static_cast<size_t>(n));
    for (Py_ssize_t i = 0; i < n; ++i) {
        try {
            r[static_cast<size_t>(i)] = position(PySequence_Fast_GET_ITEM(s, i));
        } catch (...) {
            Py_DECREF(s);
            throw;
        }
    }
    Py_DECREF(s);
    return r;
}

// x, positions, codes, params, clip_ratio, rotate
PyObject* kv4_append_batched(Args a)
{
    const Tensor& x = tensor(a[0], "x");
    heads_of(x, "x must be contiguous [B, H, 128]");
    const int B = narrow(x.size(0)), H = narrow(x.size(1));
    const std::vector<int> pos = integers(a[1]);
    require(static_cast<int>(pos.size()) == B, "one position per sequence");
    const Cache c = cache(a[2], a[3], x.size(0) * x.size(1), -1, "codes", "params",
                          "codes must be uint8 [B*H, S_max, 64] and params uint8 [B*H, S_max, 4], contiguous");
    const float ratio = real(a[4]);
    const int rotate = truth(a[5]);
    const rcp_dtype xd = in_dtype(x, kXType);
    void* const xp = dev(x, "x");
    call([&](void* st) { return rcp_kv4_append_batched(xp, xd, B, H, c.S_max, pos.data(), rotate, ratio, c.codes, c.params, st); });
    return nothing();
}

// q, lengths, k_codes, k_params, v_codes, v_params, softmax_scale, out, out_dtype, workspace
PyObject* kv4_attn_decode_batched(Args a)
{
    const Tensor& q = tensor(a[0], "q");
    heads_of(q, "q must be contiguous [B, H_q, 128]");
    const int B = narrow(q.size(0)), H_q = narrow(q.size(1));
    const char* const each = "one length per sequence, and a pooled cache of B * H_kv heads";
    const std::vector<int> lens = integers(a[1]);
    require(static_cast<int>(lens.size()) == B && B > 0, each);
    const Cache k = cache(a[2], a[3], -1, -1, "k_codes", "k_params", kPool);
    require(k.heads % B == 0, each);
    const Cache v = cache(a[4], a[5], k.heads, k.S_max, "v_codes", "v_params", kPool);
    const float scale = real(a[6]);
    const int64_t values = static_cast<int64_t>(B) * H_q * D;
    const Result out = output(a[7], a[8], {B, H_q, D}, q);
    const rcp_dtype od = out_code(out.t, "out must be float16 or float32 [B, H_q, 128]");
    require(out.t.numel() >= values, "out must be float16 or float32 [B, H_q, 128]");
    Tensor work;
    if (none(a[9])) {
        int most = 0;
        for (int n : lens) most = n > most ? n : most;
        const int64_t need = static_cast<int64_t>(B) * static_cast<int64_t>(rcp_kv4_workspace_bytes(H_q, most));
        work = empty_like_device({need > 16 ? need : 16}, at::kByte, q);
    } else
        work = tensor(a[9], "workspace");
    const rcp_dtype qd = in_dtype(q, "q must be float16, bfloat16 or float32");
    void *const qp = dev(q, "q"), *const o = dev(out.t, "out"), *const ws = dev(work, "workspace");
    const int H_kv = k.heads / B;
    call([&](void* st) {
        return rcp_kv4_attn_decode_batched(qp, qd, B, H_q, H_kv, k.S_max, lens.data(), k.codes, k.params, v.codes, v.params, scale,
                                           o, od, ws, work.nbytes(), st);
    });
    return out.give();
}

// ---- module ---------------------------------------------------------------------------------------------
template <PyObject* (*F)(Args), int COUNT>
PyObject* entry(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    if (n != COUNT) {
        PyErr_Format(PyExc_TypeError, "%d arguments wanted, %zd given", COUNT, n);
        return nullptr;
    }
    try {
        return F(a);
    } catch (const Raised&) {
    } catch (const Bad& e) {
        PyErr_SetString(PyExc_ValueError, e.what.c_str());
    } catch (const Status& e) {
        PyObject* x = PyObject_CallFunction(g_error, "is", e.rc, rcp_last_error());
        if (x != nullptr) {
            PyErr_SetObject(g_error, x);
            Py_DECREF(x);
        }
    } catch (const std::exception& e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
    }
    return nullptr;
}

PyObject* set_error(PyObject*, PyObject* type)
{
    Py_INCREF(type);
    Py_XDECREF(g_error);
    g_error = type;
    return nothing();
}

#define RCP_ENTRY(name, count) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&entry<&name, count>)), METH_FASTCALL, nullptr}
PyMethodDef g_methods[] = {
    RCP_ENTRY(w2a4_gemv, 11),
    RCP_ENTRY(rotate_quant_w2a4_gemv, 13),
    RCP_ENTRY(quant_w2a4_gemv_grouped, 13),
    RCP_ENTRY(w2a4_gemv_grouped, 11),
    RCP_ENTRY(w2a4_gemm_grouped, 12),
    RCP_ENTRY(w2a16_gemv, 7),
    RCP_ENTRY(w3a4_gemv, 10),
    RCP_ENTRY(quant_w3a4_gemv, 12),
    RCP_ENTRY(rotate_quant_act, 6),
    RCP_ENTRY(rotate_quant_act_static, 5),
    RCP_ENTRY(rotate_act, 3),
    RCP_ENTRY(pack_weights, 6),
    RCP_ENTRY(pack_weights_grouped, 7),
    RCP_ENTRY(pack_weights_w3, 7),
    RCP_ENTRY(kv4_append, 6),
    RCP_ENTRY(kv4_append_kv, 9),
    RCP_ENTRY(kv4_attn_decode, 11),
    RCP_ENTRY(kv4_append_batched, 6),
    RCP_ENTRY(kv4_attn_decode_batched, 10),
    {"set_error", set_error, METH_O, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
#undef RCP_ENTRY

PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_rcp_host", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__rcp_host() { return PyModule_Create(&g_module); }
