// Python binding of the C ABI (include/fp8mm.h) for torch tensors: argument marshalling only.
//
// For the short calls of the path (a cast of a small tensor is 3 us of GPU time) the host side is what
// counts: marshalling eighteen arguments through ctypes and asking tensors for their properties from
// Python took 5 - 9 us a call.  Here the arguments are unpacked in C: under 1 us a call in front of
// the launches themselves.  Names, argument names, defaults, checks and exceptions are those of the
// documented Python functions; the GIL is released around the library call.
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <stdio.h>
#include <string.h>

#include "fp8mm.h"

namespace {

PyObject* g_error = nullptr;             // Fp8Error(status, message)

struct Failed {};                        // a Python exception is set

[[noreturn]] void raise(PyObject* type, const char* fmt, const char* a = "", const char* b = "")
{
    PyErr_Format(type, fmt, a, b);
    throw Failed{};
}

// The arguments of one call, by position or by name, in the order of `names`.
constexpr int kMost = 18;
struct Args {
    PyObject* v[kMost] = {};
    Args(const char* fn, const char* const* names, int count, int required, PyObject* const* args, Py_ssize_t nargs, PyObject* kw)
    {
        if (nargs > count) {
            PyErr_Format(PyExc_TypeError, "%s() takes at most %d arguments (%zd given)", fn, count, nargs);
            throw Failed{};
        }
        for (Py_ssize_t i = 0; i < nargs; ++i) v[i] = args[i];
        const Py_ssize_t nkw = kw ? PyTuple_GET_SIZE(kw) : 0;
        for (Py_ssize_t k = 0; k < nkw; ++k) {
            PyObject* name = PyTuple_GET_ITEM(kw, k);
            int at = 0;
            while (at < count && PyUnicode_CompareWithASCIIString(name, names[at]) != 0) ++at;
            if (at == count || v[at]) {
                PyErr_Format(PyExc_TypeError, at == count ? "%s() got an unexpected keyword argument '%U'" : "%s() got multiple values for argument '%U'", fn, name);
                throw Failed{};
            }
            v[at] = args[nargs + k];
        }
        for (int i = 0; i < required; ++i)
            if (!v[i]) raise(PyExc_TypeError, "%s() missing required argument '%s'", fn, names[i]);
    }
    PyObject* operator[](int i) const { return v[i]; }
};

bool is_none(PyObject* o) { return !o || o == Py_None; }
bool is_tensor(PyObject* o) { return o && THPVariable_Check(o); }

const at::Tensor& tensor(PyObject* o, const char* what)
{
    if (!is_tensor(o)) raise(PyExc_TypeError, "%s must be a tensor", what);
    return THPVariable_Unpack(o);
}

// The low 64 bits of an integer (or of what stands for one by __index__).
unsigned long long low_bits(PyObject* o)
{
    const unsigned long long x = PyLong_AsUnsignedLongLongMask(o);
    if (x == ~0ull && PyErr_Occurred()) throw Failed{};
    return x;
}

// The same of int(o), for arguments that anything with an integer value may be given for.
unsigned long long low_bits_of_int(PyObject* o)
{
    if (PyLong_CheckExact(o)) return low_bits(o);
    PyObject* i = PyNumber_Long(o);
    if (!i) throw Failed{};
    const unsigned long long x = PyLong_AsUnsignedLongLongMask(i);
    Py_DECREF(i);
    return x;
}

// Arguments that the C ABI takes as an int (and checks): a format; a number of slices, flags, a kind (absent: 0).
int small(PyObject* o) { return (int)low_bits(o); }
int small_of_int(PyObject* o) { return o ? (int)low_bits_of_int(o) : 0; }

int truth(PyObject* o)
{
    const int t = PyObject_IsTrue(o);
    if (t < 0) throw Failed{};
    return t;
}

// float(o)
float real(PyObject* o)
{
    PyObject* f = PyNumber_Float(o);
    if (!f) throw Failed{};
    const double d = PyFloat_AS_DOUBLE(f);
    Py_DECREF(f);
    return (float)d;
}

// None: torch's current stream; an object with a cuda_stream, or what int() makes the handle itself.
void* stream_of(PyObject* o)
{
    if (is_none(o)) return (void*)c10::hip::getCurrentHIPStream().stream();
    if (PyLong_CheckExact(o)) return (void*)(uintptr_t)low_bits(o);
    PyObject* h = PyObject_GetAttrString(o, "cuda_stream");
    if (!h) {
        if (!PyErr_ExceptionMatches(PyExc_AttributeError)) throw Failed{};
        PyErr_Clear();
        return (void*)(uintptr_t)low_bits_of_int(o);
    }
    const unsigned long long p = PyLong_AsUnsignedLongLongMask(h);
    Py_DECREF(h);
    if (p == ~0ull && PyErr_Occurred()) throw Failed{};
    return (void*)(uintptr_t)p;
}

void check_device(const at::Tensor& t, const char* what)
{
    if (!t.is_cuda()) raise(PyExc_ValueError, "%s must live in device memory", what);
    if (!t.is_contiguous()) raise(PyExc_ValueError, "%s must be contiguous", what);
}

// A tensor that is read ...
const void* device(const at::Tensor& t, const char* what) { check_device(t, what); return t.const_data_ptr(); }
const void* device(PyObject* o, const char* what) { return device(tensor(o, what), what); }
const void* device_or_null(const at::Tensor& t, const char* what) { return t.numel() ? device(t, what) : nullptr; }
const void* device_or_none(PyObject* o, const char* what) { return is_none(o) ? nullptr : device(o, what); }

// ... and one that is written: a lazy clone gets memory of its own first.
void* written(const at::Tensor& t, const char* what) { check_device(t, what); return t.mutable_data_ptr(); }
void* written(PyObject* o, const char* what) { return written(tensor(o, what), what); }
void* written_or_null(const at::Tensor& t, const char* what) { return t.numel() ? written(t, what) : nullptr; }
void* written_or_none(PyObject* o, const char* what) { return is_none(o) ? nullptr : written(o, what); }

int dtype_of(const at::Tensor& t)
{
    if (t.scalar_type() == at::kFloat) return FP8_F32;
    if (t.scalar_type() == at::kBFloat16) return FP8_BF16;
    raise(PyExc_TypeError, "expected a float32 or bfloat16 tensor, got %s", c10::toString(t.scalar_type()));
}

// fp32 cells on the device: `count` of them (-1: any number).
const at::Tensor& cells_tensor(PyObject* o, const char* what, int64_t count)
{
    const at::Tensor& t = tensor(o, what);
    if (t.scalar_type() != at::kFloat || (count >= 0 && t.numel() != count)) {
        if (count < 0) raise(PyExc_ValueError, "%s must be an fp32 device tensor", what);
        PyErr_Format(PyExc_ValueError, "%s must be an fp32 device tensor of %lld values", what, (long long)count);
        throw Failed{};
    }
    return t;
}
const float* cells(PyObject* o, const char* what, int64_t count) { return (const float*)device(cells_tensor(o, what, count), what); }
float* cells_out(PyObject* o, const char* what, int64_t count) { return (float*)written(cells_tensor(o, what, count), what); }

bool is_bytes(const at::Tensor& t) { return t.scalar_type() == at::kByte; }

// FP8 bytes for the elements of x
uint8_t* bytes_for(PyObject* o, const at::Tensor& x)
{
    const at::Tensor& q = tensor(o, "q_out");
    if (!is_bytes(q) || q.numel() != x.numel()) raise(PyExc_ValueError, "q_out must be uint8 with as many elements as x");
    return (uint8_t*)(x.numel() ? written(q, "q_out") : nullptr);
}

void workspace_holds(const at::Tensor& ws, int tensors, const char* text)
{
    if (ws.numel() * (int64_t)ws.element_size() < (int64_t)tensors * FP8_AMAX_WORKSPACE_BYTES) raise(PyExc_ValueError, "%s", text);
}

template <class F>
PyObject* checked(F call)
{
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = call();
    Py_END_ALLOW_THREADS
    if (status == FP8_OK) Py_RETURN_NONE;
    if (PyObject* e = PyObject_CallFunction(g_error, "is", status, fp8_last_error())) {
        PyErr_SetObject(g_error, e);
        Py_DECREF(e);
    }
    return nullptr;
}

template <class F>
PyObject* guarded(F body)
{
    try {
        return body();
    } catch (const Failed&) {
        return nullptr;
    } catch (const std::exception& e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
}

#define ENTRY(NAME, REQUIRED, ...)                                                                     \
    PyObject* NAME##_body(const Args& a);                                                              \
    PyObject* py_##NAME(PyObject*, PyObject* const* args, Py_ssize_t nargs, PyObject* kw)              \
    {                                                                                                  \
        static const char* const names[] = {__VA_ARGS__};                                              \
        return guarded([&] { return NAME##_body(Args(#NAME, names, sizeof names / sizeof *names, REQUIRED, args, nargs, kw)); }); \
    }                                                                                                  \
    PyObject* NAME##_body(const Args& a)

ENTRY(fp8_amax, 2, "x", "amax_out", "stream")
{
    const at::Tensor& x = tensor(a[0], "x");
    const void* p = device_or_null(x, "x");
    const int dt = dtype_of(x);
    float* out = (float*)written(a[1], "amax_out");
    void* s = stream_of(a[2]);
    const size_t n = (size_t)x.numel();
    return checked([&] { return ::fp8_amax(p, n, dt, out, s); });
}

ENTRY(fp8_amax_scale, 5, "x", "fmt", "amax_out", "scale_out", "workspace", "stream")
{
    const at::Tensor& ws = tensor(a[4], "workspace");
    workspace_holds(ws, 1, "workspace must hold FP8_AMAX_WORKSPACE_BYTES bytes");
    const at::Tensor& x = tensor(a[0], "x");
    const void* p = device_or_null(x, "x");
    const int dt = dtype_of(x), fmt = small(a[1]);
    float *amax = (float*)written(a[2], "amax_out"), *scale = (float*)written_or_none(a[3], "scale_out");
    void *w = written(ws, "workspace"), *s = stream_of(a[5]);
    const size_t n = (size_t)x.numel();
    return checked([&] { return ::fp8_amax_scale(p, n, dt, fmt, amax, scale, w, s); });
}

// A sequence as a list or tuple, released at the end.
struct Sequence {
    PyObject* s;
    Sequence(PyObject* o, const char* what) : s(PySequence_Fast(o, what)) { if (!s) throw Failed{}; }
    ~Sequence() { Py_DECREF(s); }
    Py_ssize_t size() const { return PySequence_Fast_GET_SIZE(s); }
    PyObject* operator[](Py_ssize_t i) const { return PySequence_Fast_GET_ITEM(s, i); }
};

// The host-side argument arrays of the multi-tensor entry points: device pointers, element counts, formats.
struct Tensors {
    int count = 0, dtype = FP8_BF16;
    const void* x[FP8_MULTI_MAX];
    size_t n[FP8_MULTI_MAX];
    int fmt[FP8_MULTI_MAX];
    Tensors(const Sequence& xs, PyObject* fmts, const char* who)
    {
        const Sequence f(fmts, "fmts must be a sequence");
        if (xs.size() > FP8_MULTI_MAX || f.size() != xs.size()) {
            PyErr_Format(PyExc_ValueError, "%s: at most %d tensors, one format each", who, FP8_MULTI_MAX);
            throw Failed{};
        }
        count = (int)xs.size();
        for (int i = 0; i < count; ++i) {
            const at::Tensor& t = tensor(xs[i], "x");
            const int dt = dtype_of(t);
            if (i && dt != dtype) raise(PyExc_TypeError, "%s: all tensors must have one element type", who);
            dtype = dt;
            x[i] = device_or_null(t, "x");
            n[i] = (size_t)t.numel();
            fmt[i] = small_of_int(f[i]);
        }
    }
};

ENTRY(fp8_amax_scale_multi, 5, "xs", "fmts", "amax_out", "scale_out", "workspace", "stream")
{
    const Sequence xs(a[0], "xs must be a sequence of tensors");
    const Tensors t(xs, a[1], "fp8_amax_scale_multi");
    const at::Tensor& ws = tensor(a[4], "workspace");
    workspace_holds(ws, t.count, "workspace must hold FP8_AMAX_WORKSPACE_BYTES bytes per tensor");
    float *amax = cells_out(a[2], "amax_out", t.count), *scale = is_none(a[3]) ? nullptr : cells_out(a[3], "scale_out", t.count);
    void *w = written(ws, "workspace"), *s = stream_of(a[5]);
    return checked([&] { return ::fp8_amax_scale_multi(t.count, t.x, t.n, t.dtype, t.fmt, amax, scale, w, s); });
}

ENTRY(fp8_quantize_multi, 4, "xs", "fmts", "scale", "q_outs", "stream")
{
    const Sequence xs(a[0], "xs must be a sequence of tensors"), qs(a[3], "q_outs must be a sequence of tensors");
    const Tensors t(xs, a[1], "fp8_quantize_multi");
    uint8_t* q[FP8_MULTI_MAX];
    bool fine = qs.size() == t.count;
    for (int i = 0; fine && i < t.count; ++i) {
        const at::Tensor& o = tensor(qs[i], "q_out");
        fine = is_bytes(o) && (size_t)o.numel() == t.n[i];
        if (fine) q[i] = (uint8_t*)written_or_null(o, "q_out");
    }
    if (!fine) raise(PyExc_ValueError, "q_outs must be uint8 tensors with as many elements as their inputs");
    const float* scale = cells(a[2], "scale", t.count);
    void* s = stream_of(a[4]);
    return checked([&] { return ::fp8_quantize_multi(t.count, t.x, t.n, t.dtype, t.fmt, scale, q, s); });
}

ENTRY(fp8_scale_from_amax, 3, "amax", "fmt", "scale_out", "stream")
{
    const float* amax = (const float*)device(a[0], "amax");
    float* out = (float*)written(a[2], "scale_out");
    const int fmt = small(a[1]);
    void* s = stream_of(a[3]);
    return checked([&] { return ::fp8_scale_from_amax(amax, fmt, out, s); });
}

ENTRY(fp8_quantize, 4, "x", "fmt", "scale", "q_out", "stream")
{
    const at::Tensor& x = tensor(a[0], "x");
    uint8_t* q = bytes_for(a[3], x);
    const void* p = device_or_null(x, "x");
    const int dt = dtype_of(x), fmt = small(a[1]);
    const float scale = real(a[2]);
    void* s = stream_of(a[4]);
    const size_t n = (size_t)x.numel();
    return checked([&] { return ::fp8_quantize(p, n, dt, fmt, scale, q, s); });
}

ENTRY(fp8_quantize_dscale, 4, "x", "fmt", "scale", "q_out", "stream")
{
    const at::Tensor& x = tensor(a[0], "x");
    uint8_t* q = bytes_for(a[3], x);
    const void* p = device_or_null(x, "x");
    const int dt = dtype_of(x), fmt = small(a[1]);
    const float* scale = (const float*)device(a[2], "scale");
    void* s = stream_of(a[4]);
    const size_t n = (size_t)x.numel();
    return checked([&] { return ::fp8_quantize_dscale(p, n, dt, fmt, scale, q, s); });
}

// A factor given as a number or as a device tensor.
struct Factor {
    float host = 0.0f;
    const float* dev = nullptr;
    Factor(PyObject* o, const char* what, bool one_cell = false)
    {
        if (!is_tensor(o)) host = real(o);
        else dev = one_cell ? cells(o, what, 1) : (const float*)device(o, what);
    }
};

ENTRY(fp8_quantize_ex, 5, "x", "fmt", "scale", "flags", "q_out", "stream")
{
    const at::Tensor& x = tensor(a[0], "x");
    uint8_t* q = bytes_for(a[4], x);
    const void* p = device_or_null(x, "x");
    const int dt = dtype_of(x), fmt = small(a[1]), flags = small_of_int(a[3]);
    const Factor f(a[2], "scale");
    void* s = stream_of(a[5]);
    const size_t n = (size_t)x.numel();
    return checked([&] { return ::fp8_quantize_ex(p, n, dt, fmt, f.host, f.dev, flags, q, s); });
}

ENTRY(fp8_dequantize, 4, "q", "fmt", "scale", "out", "stream")
{
    const at::Tensor &q = tensor(a[0], "q"), &out = tensor(a[3], "out");
    if (!is_bytes(q) || out.numel() != q.numel()) raise(PyExc_ValueError, "q must be uint8 and out must have as many elements");
    const uint8_t* p = (const uint8_t*)device_or_null(q, "q");
    const Factor f(a[2], "scale");
    const int dt = dtype_of(out), fmt = small(a[1]);
    void *o = q.numel() ? written(out, "out") : nullptr, *s = stream_of(a[4]);
    const size_t n = (size_t)q.numel();
    return checked([&] { return ::fp8_dequantize(p, n, fmt, f.host, f.dev, dt, o, s); });
}

ENTRY(fp8_quantize_amax, 5, "x", "fmt", "scale", "q_out", "amax_out", "stream")
{
    const at::Tensor& x = tensor(a[0], "x");
    uint8_t* q = bytes_for(a[3], x);
    const void* p = device_or_null(x, "x");
    const int dt = dtype_of(x), fmt = small(a[1]);
    const float* scale = cells(a[2], "scale", 1);
    float* amax = cells_out(a[4], "amax_out", 1);
    void* s = stream_of(a[5]);
    const size_t n = (size_t)x.numel();
    return checked([&] { return ::fp8_quantize_amax(p, n, dt, fmt, scale, q, amax, s); });
}

ENTRY(fp8_quantize_sr, 5, "x", "fmt", "scale", "seed", "q_out", "stream")
{
    const at::Tensor& x = tensor(a[0], "x");
    uint8_t* q = bytes_for(a[4], x);
    const void* p = device_or_null(x, "x");
    const int dt = dtype_of(x), fmt = small(a[1]);
    Factor f(a[2], "scale", true);
    if (f.dev) f.host = 1.0f;
    const unsigned long long seed = low_bits_of_int(a[3]);
    void* s = stream_of(a[5]);
    const size_t n = (size_t)x.numel();
    return checked([&] { return ::fp8_quantize_sr(p, n, dt, fmt, f.host, f.dev, seed, q, s); });
}

ENTRY(fp8_scale_from_amax_history, 3, "amax_history", "fmt", "scale_out", "stream")
{
    const at::Tensor& h = tensor(a[0], "amax_history");
    const float* p = h.numel() ? cells(a[0], "amax_history", -1) : nullptr;
    float* out = cells_out(a[2], "scale_out", 1);
    const int fmt = small(a[1]);
    void* s = stream_of(a[3]);
    const size_t n = (size_t)h.numel();
    return checked([&] { return ::fp8_scale_from_amax_history(p, n, fmt, out, s); });
}

ENTRY(fp8_scale_from_amax_n, 3, "amax", "fmt", "scale_out", "stream")
{
    const int64_t n = tensor(a[0], "amax").numel();
    const float* p = n ? cells(a[0], "amax", -1) : nullptr;
    float* out = n ? cells_out(a[2], "scale_out", n) : nullptr;
    const int fmt = small(a[1]);
    void* s = stream_of(a[3]);
    return checked([&] { return ::fp8_scale_from_amax_n(p, (size_t)n, fmt, out, s); });
}

void matrix(const at::Tensor& x, const char* what)
{
    if (x.dim() != 2) raise(PyExc_ValueError, "%s must be a 2-D tensor", what);
}

bool has_shape(const at::Tensor& t, int64_t rows, int64_t cols) { return t.dim() == 2 && t.size(0) == rows && t.size(1) == cols; }

ENTRY(fp8_amax_rows, 2, "x", "amax_out", "stream")
{
    const at::Tensor& x = tensor(a[0], "x");
    matrix(x, "x");
    const int64_t rows = x.size(0), cols = x.size(1);
    const void* p = device_or_null(x, "x");
    const int dt = dtype_of(x);
    float* amax = rows ? cells_out(a[1], "amax_out", rows) : nullptr;
    void* s = stream_of(a[2]);
    return checked([&] { return ::fp8_amax_rows(p, rows, cols, dt, amax, s); });
}

ENTRY(fp8_quantize_rows, 4, "x", "fmt", "scale", "q_out", "stream")
{
    const at::Tensor &x = tensor(a[0], "x"), &q = tensor(a[3], "q_out");
    matrix(x, "x");
    const int64_t rows = x.size(0), cols = x.size(1);
    if (!is_bytes(q) || !has_shape(q, rows, cols)) raise(PyExc_ValueError, "q_out must be a uint8 tensor of the shape of x");
    const bool work = x.numel() > 0;
    const void* p = device_or_null(x, "x");
    const int dt = dtype_of(x), fmt = small(a[1]);
    const float* scale = work ? cells(a[2], "scale", rows) : nullptr;
    uint8_t* o = (uint8_t*)written_or_null(q, "q_out");
    void* s = stream_of(a[4]);
    return checked([&] { return ::fp8_quantize_rows(p, rows, cols, dt, fmt, scale, o, s); });
}

ENTRY(fp8_quantize_transpose, 5, "x", "fmt", "scale", "q_out", "qt_out", "stream")
{
    const at::Tensor &x = tensor(a[0], "x"), &qt = tensor(a[4], "qt_out");
    matrix(x, "x");
    const int64_t rows = x.size(0), cols = x.size(1);
    if (!is_bytes(qt) || !has_shape(qt, cols, rows)) raise(PyExc_ValueError, "qt_out must be a uint8 tensor of shape (cols, rows)");
    const bool work = x.numel() > 0;
    uint8_t* q = nullptr;
    if (!is_none(a[3])) {
        const at::Tensor& t = tensor(a[3], "q_out");
        if (!is_bytes(t) || !has_shape(t, rows, cols)) raise(PyExc_ValueError, "q_out must be None or a uint8 tensor of the shape of x");
        q = (uint8_t*)written_or_null(t, "q_out");
    }
    const void* p = device_or_null(x, "x");
    const int dt = dtype_of(x), fmt = small(a[1]);
    const float* scale = work ? cells(a[2], "scale", 1) : nullptr;
    uint8_t* t = (uint8_t*)written_or_null(qt, "qt_out");
    void* s = stream_of(a[5]);
    return checked([&] { return ::fp8_quantize_transpose(p, rows, cols, dt, fmt, scale, q, t, s); });
}

// The operands and the output of a product: FP8 bytes (or, `wide`, tensors of one wider type) and their shapes.
struct Product {
    const uint8_t *A, *B;
    void* C;
    int64_t M, N, K;
    Product(const at::Tensor& ta, bool transA, const at::Tensor& tb, bool transB, const at::Tensor& tc, const char* names, const char* shapes,
            bool bytes = true)
    {
        if (ta.dim() != 2 || tb.dim() != 2 || (bytes && (!is_bytes(ta) || !is_bytes(tb)))) raise(PyExc_ValueError, "%s", names);
        M = ta.size(transA ? 1 : 0); K = ta.size(transA ? 0 : 1);
        N = tb.size(transB ? 0 : 1);
        if (tb.size(transB ? 1 : 0) != K || !has_shape(tc, M, N)) raise(PyExc_ValueError, "%s", shapes);
        A = (const uint8_t*)device_or_null(ta, "A");
        B = (const uint8_t*)device_or_null(tb, "B");
        C = written_or_null(tc, "C");
    }
};
const char* const kBytes2d = "A and B must be 2-D uint8 tensors of FP8 bytes";
const char* const kShapesEx = "shapes do not form C[M,N] = op(A)[M,K] op(B)[K,N]";

template <class F>
PyObject* plain_gemm(const Args& a, F call)
{
    const at::Tensor& c = tensor(a[6], "C");
    const Product p(tensor(a[0], "A"), false, tensor(a[3], "B"), false, c, kBytes2d, "shapes do not form C[M,N] = A[M,K] B[K,N]");
    const int fa = small(a[1]), fb = small(a[4]), dt = dtype_of(c);
    void* s = stream_of(a[7]);
    return checked([&] { return call(p, fa, fb, dt, s); });
}

#define PLAIN_GEMM(NAME, GET)                                                                                           \
    ENTRY(NAME, 7, "A", "fmtA", "sA", "B", "fmtB", "sB", "C", "stream")                                                 \
    {                                                                                                                   \
        const auto sA = GET(a[2], "sA"), sB = GET(a[5], "sB");                                                          \
        return plain_gemm(a, [=](const Product& p, int fa, int fb, int dt, void* s) {                                   \
            return ::NAME(p.A, fa, sA, p.B, fb, sB, p.C, p.M, p.N, p.K, dt, s); });                                     \
    }
float by_value(PyObject* o, const char*) { return real(o); }
const float* on_device(PyObject* o, const char* what) { return (const float*)device(o, what); }
PLAIN_GEMM(fp8_gemm, by_value)
PLAIN_GEMM(fp8_gemm_mfma8, by_value)
PLAIN_GEMM(fp8_gemm_dscale, on_device)
PLAIN_GEMM(fp8_gemm_mfma8_dscale, on_device)

// sA and sB: both numbers or both device tensors.
struct Factors {
    Factor A, B;
    Factors(PyObject* a, PyObject* b) : A(a, "sA"), B(b, "sB")
    {
        if (is_tensor(a) != is_tensor(b)) raise(PyExc_ValueError, "sA and sB must both be floats or both device tensors");
    }
};

ENTRY(fp8_gemm_ex, 9, "A", "fmtA", "transA", "B", "fmtB", "transB", "C", "sA", "sB", "flags", "stream")
{
    const int tA = truth(a[2]), tB = truth(a[5]);
    const at::Tensor& c = tensor(a[6], "C");
    const Product p(tensor(a[0], "A"), tA, tensor(a[3], "B"), tB, c, kBytes2d, kShapesEx);
    const Factors f(a[7], a[8]);
    const int fa = small(a[1]), fb = small(a[4]), dt = dtype_of(c), flags = small_of_int(a[9]);
    void* s = stream_of(a[10]);
    return checked([&] { return ::fp8_gemm_ex(p.A, fa, tA, p.B, fb, tB, p.C, p.M, p.N, p.K, dt, f.A.host, f.B.host, f.A.dev, f.B.dev, flags, s); });
}

ENTRY(fp8_gemm_splitk, 10, "A", "fmtA", "transA", "B", "fmtB", "transB", "C", "sA", "sB", "workspace", "flags", "splits", "stream")
{
    const int tA = truth(a[2]), tB = truth(a[5]);
    const at::Tensor& c = tensor(a[6], "C");
    const Product p(tensor(a[0], "A"), tA, tensor(a[3], "B"), tB, c, kBytes2d, kShapesEx);
    const Factors f(a[7], a[8]);
    const int fa = small(a[1]), fb = small(a[4]), dt = dtype_of(c), flags = small_of_int(a[10]), splits = small_of_int(a[11]);
    void *ws = written_or_none(a[9], "workspace"), *s = stream_of(a[12]);
    const size_t bytes = is_none(a[9]) ? 0 : (size_t)tensor(a[9], "workspace").numel() * tensor(a[9], "workspace").element_size();
    return checked([&] { return ::fp8_gemm_splitk(p.A, fa, tA, p.B, fb, tB, p.C, p.M, p.N, p.K, dt, f.A.host, f.B.host, f.A.dev, f.B.dev, flags, splits,
                                                  ws, bytes, s); });
}

ENTRY(fp8_gemm_splitk_static, 9, "A", "fmtA", "transA", "B", "fmtB", "transB", "C", "sA", "sB", "flags", "splits", "stream")
{
    const int tA = truth(a[2]), tB = truth(a[5]);
    const at::Tensor& c = tensor(a[6], "C");
    const Product p(tensor(a[0], "A"), tA, tensor(a[3], "B"), tB, c, kBytes2d, kShapesEx);
    const Factors f(a[7], a[8]);
    const int fa = small(a[1]), fb = small(a[4]), dt = dtype_of(c), flags = small_of_int(a[9]), splits = small_of_int(a[10]);
    void* s = stream_of(a[11]);
    return checked([&] { return ::fp8_gemm_splitk_static(p.A, fa, tA, p.B, fb, tB, p.C, p.M, p.N, p.K, dt, f.A.host, f.B.host, f.A.dev, f.B.dev, flags,
                                                         splits, s); });
}

ENTRY(fp8_gemm_fused, 10, "A", "fmtA", "transA", "B", "fmtB", "transB", "D", "out_kind", "sA", "sB", "sD", "amax_out", "flags", "stream")
{
    const int tA = truth(a[2]), tB = truth(a[5]), kind = small_of_int(a[7]);
    const at::Tensor &d = tensor(a[6], "D"), &sA = tensor(a[8], "sA"), &sB = tensor(a[9], "sB");
    const Product p(tensor(a[0], "A"), tA, tensor(a[3], "B"), tB, d, kBytes2d, "shapes do not form D[M,N] = op(A)[M,K] op(B)[K,N]");
    const at::ScalarType want = kind == FP8_OUT_F32 ? at::kFloat : kind == FP8_OUT_BF16 ? at::kBFloat16 : at::kByte;
    if (d.scalar_type() != want) {
        PyErr_Format(PyExc_ValueError, "D must be %s for out_kind %d", c10::toString(want), kind);
        throw Failed{};
    }
    static const char* const names[] = {"sA", "sB", "sD", "amax_out"};
    for (int i = 0; i < 4; ++i)
        if (!is_none(a[8 + i]) && tensor(a[8 + i], names[i]).scalar_type() != at::kFloat) raise(PyExc_ValueError, "%s must be an fp32 device tensor", names[i]);
    const float *pA = (const float*)device(sA, "sA"), *pB = (const float*)device(sB, "sB"), *pD = (const float*)device_or_none(a[10], "sD");
    float* amax = (float*)written_or_none(a[11], "amax_out");
    const int fa = small(a[1]), fb = small(a[4]), flags = small_of_int(a[12]);
    const int64_t nA = sA.numel(), nB = sB.numel();
    void* s = stream_of(a[13]);
    return checked([&] { return ::fp8_gemm_fused(p.A, fa, tA, p.B, fb, tB, p.C, kind, p.M, p.N, p.K, pA, nA, pB, nB, pD, amax, flags, s); });
}

ENTRY(fp8_scaled_gemm, 12, "a", "fmtA", "transA", "b", "fmtB", "transB", "qa_out", "qb_out", "amax_out", "scale_out", "workspace", "C", "flags", "stream")
{
    const int tA = truth(a[2]), tB = truth(a[5]);
    const at::Tensor &x = tensor(a[0], "a"), &y = tensor(a[3], "b"), &c = tensor(a[11], "C"), &ws = tensor(a[10], "workspace");
    const char* const operands = "a and b must be 2-D tensors of one element type";
    if (x.scalar_type() != y.scalar_type()) raise(PyExc_ValueError, "%s", operands);
    const Product p(x, tA, y, tB, c, operands, "shapes do not form C[M,N] = op(a)[M,K] op(b)[K,N]", false);
    const at::Tensor &qx = tensor(a[6], "qa_out"), &qy = tensor(a[7], "qb_out");
    if (!is_bytes(qx) || qx.sizes() != x.sizes() || !is_bytes(qy) || qy.sizes() != y.sizes())
        raise(PyExc_ValueError, "qa_out / qb_out must be uint8 tensors of the operands' shapes");
    workspace_holds(ws, 2, "workspace must hold 2 * FP8_AMAX_WORKSPACE_BYTES bytes");
    const int dt = dtype_of(x), odt = dtype_of(c), fa = small(a[1]), fb = small(a[4]), flags = small_of_int(a[12]);
    uint8_t *qa = (uint8_t*)written_or_null(qx, "qa_out"), *qb = (uint8_t*)written_or_null(qy, "qb_out");
    float *amax = cells_out(a[8], "amax_out", 2), *scale = cells_out(a[9], "scale_out", 2);
    void *w = written(ws, "workspace"), *s = stream_of(a[13]);
    return checked([&] { return ::fp8_scaled_gemm(p.A, p.B, dt, tA, tB, p.M, p.N, p.K, fa, fb, qa, qb, amax, scale, w, p.C, odt, flags, s); });
}

// Called once by the package: the exception that failing calls raise.
PyObject* py_set_error(PyObject*, PyObject* type)
{
    Py_INCREF(type);
    Py_XDECREF(g_error);
    g_error = type;
    Py_RETURN_NONE;
}

#define METHOD(NAME, DOC) {#NAME, (PyCFunction)(void (*)(void))py_##NAME, METH_FASTCALL | METH_KEYWORDS, DOC}
PyMethodDef methods[] = {
    METHOD(fp8_amax, "fp8_amax(x, amax_out, stream=None)\n--\n\n"),
    METHOD(fp8_amax_scale, "fp8_amax_scale(x, fmt, amax_out, scale_out, workspace, stream=None)\n--\n\namax and scale = fmt_max / amax in one launch; workspace: device "
           "tensor of at least\nFP8_AMAX_WORKSPACE_BYTES bytes, zero-filled once before its first use."),
    METHOD(fp8_amax_scale_multi, "fp8_amax_scale_multi(xs, fmts, amax_out, scale_out, workspace, stream=None)\n--\n\nfp8_amax_scale for up to FP8_MULTI_MAX tensors of "
           "one element type in one launch: amax_out and\nscale_out are fp32 device tensors of len(xs) values, workspace holds len(xs) * FP8_AMAX_WORKSPACE_BYTES bytes."),
    METHOD(fp8_quantize_multi, "fp8_quantize_multi(xs, fmts, scale, q_outs, stream=None)\n--\n\nfp8_quantize_dscale for up to FP8_MULTI_MAX tensors of one element type in "
           "one launch; scale is an\nfp32 device tensor of len(xs) factors, q_outs the uint8 outputs."),
    METHOD(fp8_scale_from_amax, "fp8_scale_from_amax(amax, fmt, scale_out, stream=None)\n--\n\n"),
    METHOD(fp8_quantize, "fp8_quantize(x, fmt, scale, q_out, stream=None)\n--\n\n"),
    METHOD(fp8_quantize_dscale, "fp8_quantize_dscale(x, fmt, scale, q_out, stream=None)\n--\n\n"),
    METHOD(fp8_quantize_ex, "fp8_quantize_ex(x, fmt, scale, flags, q_out, stream=None)\n--\n\n`scale` is a float or a one-element device tensor."),
    METHOD(fp8_dequantize, "fp8_dequantize(q, fmt, scale, out, stream=None)\n--\n\n`scale` is a float or a one-element device tensor; out is float32 or bfloat16."),
    METHOD(fp8_quantize_amax, "fp8_quantize_amax(x, fmt, scale, q_out, amax_out, stream=None)\n--\n\nCast x with the one-element device tensor `scale` and write max |x| into amax_out."),
    METHOD(fp8_quantize_sr, "fp8_quantize_sr(x, fmt, scale, seed, q_out, stream=None)\n--\n\nStochastic-rounding cast; scale is a float or a one-element fp32 device tensor."),
    METHOD(fp8_scale_from_amax_history, "fp8_scale_from_amax_history(amax_history, fmt, scale_out, stream=None)\n--\n\n"),
    METHOD(fp8_scale_from_amax_n, "fp8_scale_from_amax_n(amax, fmt, scale_out, stream=None)\n--\n\n"),
    METHOD(fp8_amax_rows, "fp8_amax_rows(x, amax_out, stream=None)\n--\n\n"),
    METHOD(fp8_quantize_rows, "fp8_quantize_rows(x, fmt, scale, q_out, stream=None)\n--\n\n"),
    METHOD(fp8_quantize_transpose, "fp8_quantize_transpose(x, fmt, scale, q_out, qt_out, stream=None)\n--\n\nq_out (rows x cols, may be None) and qt_out (cols x rows) "
           "receive the FP8 bytes of x."),
    METHOD(fp8_gemm, "fp8_gemm(A, fmtA, sA, B, fmtB, sB, C, stream=None)\n--\n\n"),
    METHOD(fp8_gemm_dscale, "fp8_gemm_dscale(A, fmtA, sA, B, fmtB, sB, C, stream=None)\n--\n\n"),
    METHOD(fp8_gemm_mfma8, "fp8_gemm_mfma8(A, fmtA, sA, B, fmtB, sB, C, stream=None)\n--\n\n"),
    METHOD(fp8_gemm_mfma8_dscale, "fp8_gemm_mfma8_dscale(A, fmtA, sA, B, fmtB, sB, C, stream=None)\n--\n\n"),
    METHOD(fp8_gemm_ex, "fp8_gemm_ex(A, fmtA, transA, B, fmtB, transB, C, sA, sB, flags=0, stream=None)\n--\n\nA is [M, K] (or [K, M] if transA), B is [K, N] (or [N, K] "
           "if transB); sA and sB are both\nfloats or both one-element device tensors."),
    METHOD(fp8_gemm_splitk, "fp8_gemm_splitk(A, fmtA, transA, B, fmtB, transB, C, sA, sB, workspace, flags=0, splits=0, stream=None)\n--\n\nfp8_gemm_ex with K cut into "
           "slices; `workspace` is a device tensor (any dtype) of at least\nfp8_gemm_splitk_workspace_size(...) bytes, or None where that is 0."),
    METHOD(fp8_gemm_splitk_static, "fp8_gemm_splitk_static(A, fmtA, transA, B, fmtB, transB, C, sA, sB, flags=0, splits=0, stream=None)\n--\n\nfp8_gemm_splitk with the "
           "library's own scratch array in place of a workspace; allocates nothing."),
    METHOD(fp8_gemm_fused, "fp8_gemm_fused(A, fmtA, transA, B, fmtB, transB, D, out_kind, sA, sB, sD=None, amax_out=None, flags=0, stream=None)\n--\n\nA is [M, K] (or "
           "[K, M] if transA), B is [K, N] (or [N, K] if transB), D is [M, N] of the\nelement type of out_kind (uint8 for the FP8 kinds).  sA: fp32 device tensor of 1 or "
           "M values,\nsB: of 1 or N values; sD: None or one value; amax_out: None or one fp32 cell."),
    METHOD(fp8_scaled_gemm, "fp8_scaled_gemm(a, fmtA, transA, b, fmtB, transB, qa_out, qb_out, amax_out, scale_out, workspace, C, flags=0, stream=None)\n--\n\namax + scale + "
           "cast of both operands and their FP8 product in one call.  a is [M, K] (or\n[K, M] if transA), b is [K, N] (or [N, K] if transB), both bf16 or both fp32; "
           "qa_out / qb_out are\nuint8 tensors of the operands' shapes; amax_out and scale_out hold two floats ([0]: a, [1]: b);\nworkspace: 2 * FP8_AMAX_WORKSPACE_BYTES "
           "bytes, zero-filled once."),
    {"set_error", py_set_error, METH_O, "The exception class that failing calls raise."},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_native", "C ABI entry points for torch tensors.", -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) { return PyModule_Create(&module_def); }
