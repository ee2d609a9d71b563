// The calls a model makes for every layer, as a CPython extension: torch tensors in, one C ABI call, torch tensor out.
// binding.py holds the public functions (names, defaults, documentation) and hands their arguments on in order.
//
// A small layer's kernels take less time than the interpreter needs to take five tensors apart: through ctypes one
// forward cost 14 us of host time, of which the two launches are 7 (MI355X host, M1 x N256 x K3072); here tensors are
// read as the C++ objects they are.
#include <Python.h>

#include <ATen/ops/empty.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "convrot.h"

namespace {

// The entry points, at the addresses that binding.py looked up in the library it loaded (bind): a process has one libconvrot, with
// one static workspace, wherever binding.py takes it from.
#define CONVROT_CALLS(F)                                                                                                     \
    F(convrot_packed_bytes) F(convrot_packed_bytes8) F(convrot_workspace_bytes) F(convrot_workspace_bytes8)                  \
    F(convrot_rotquant_act) F(convrot_rotquant_act8) F(convrot_w4a4_gemm_dequant) F(convrot_w8a8_gemm_dequant)               \
    F(convlinear4bit_forward) F(convlinear4bit_forward_noalloc) F(convlinear8bit_forward)
struct Library {
#define CONVROT_MEMBER(name) decltype(&::name) name;
    CONVROT_CALLS(CONVROT_MEMBER)
#undef CONVROT_MEMBER
} lib;
bool bound = false;

struct Failed {};   // a Python error is set

[[noreturn]] void fail(PyObject *type, const char *format, const char *a, long long b = 0, long long c = 0)
{
    PyErr_Format(type, format, a, b, c);
    throw Failed{};
}

const at::Tensor &tensor(PyObject *o, const char *name)
{
    if (!THPVariable_Check(o)) fail(PyExc_TypeError, "%s: need a torch tensor", name);
    return THPVariable_Unpack(o);
}

const at::Tensor &device_tensor(PyObject *o, at::ScalarType type, const char *type_name, const char *name)
{
    const at::Tensor &t = tensor(o, name);
    if (!(t.is_cuda() && t.scalar_type() == type && t.is_contiguous())) {
        PyErr_Format(PyExc_TypeError, "%s: need a contiguous %s tensor on the GPU", name, type_name);
        throw Failed{};
    }
    return t;
}

const at::Tensor &bf16(PyObject *o, const char *name) { return device_tensor(o, at::kBFloat16, "torch.bfloat16", name); }
const at::Tensor &f32(PyObject *o, const char *name) { return device_tensor(o, at::kFloat, "torch.float32", name); }

// A code matrix: an opaque uint8 buffer of at least `bytes` bytes.
const at::Tensor &codes(PyObject *o, size_t bytes, const char *name)
{
    const at::Tensor &t = device_tensor(o, at::kByte, "torch.uint8", name);
    if ((size_t)t.numel() < bytes)
        fail(PyExc_ValueError, "%s: need %lld bytes (convrot_packed_bytes), got %lld", name, (long long)bytes, (long long)t.numel());
    return t;
}

const void *bias_of(PyObject *o, int64_t N)
{
    if (o == Py_None) return nullptr;
    const at::Tensor &b = bf16(o, "bias");
    if (b.dim() != 1 || b.size(0) != N) fail(PyExc_ValueError, "%s: need shape [N]", "bias");
    return b.data_ptr();
}

void matrix(const at::Tensor &t, const char *name, int64_t &rows, int64_t &cols)
{
    if (t.dim() != 2) fail(PyExc_ValueError, "%s: need a matrix, got %lld dimensions", name, (long long)t.dim());
    rows = t.size(0);
    cols = t.size(1);
}

int64_t length(const at::Tensor &t, const char *name)
{
    if (t.dim() < 1) fail(PyExc_ValueError, "%s: need a vector, got %lld dimensions", name, (long long)t.dim());
    if (t.numel() < t.size(0)) fail(PyExc_ValueError, "%s: need a vector, got %lld elements in %lld rows", name, (long long)t.numel(), (long long)t.size(0));
    return t.size(0);
}

long long integer(PyObject *o)
{
    const long long v = PyLong_AsLongLong(o);
    if (v == -1 && PyErr_Occurred()) throw Failed{};
    return v;
}

void *stream_of(PyObject *o)
{
    if (o == Py_None) return c10::hip::getCurrentHIPStream().stream();
    PyObject *s = PyObject_GetAttrString(o, "cuda_stream");
    if (!s) throw Failed{};
    void *p = PyLong_AsVoidPtr(s);
    Py_DECREF(s);
    if (!p && PyErr_Occurred()) throw Failed{};
    return p;
}

// A tensor that a call on `stream` writes.  Where that is not torch's current stream the memory has to be the call's stream's own:
// torch hands memory that is freed on a stream to that stream's next tensors at once, so a block of the current stream's may
// still be in use there when the call writes it, and one that is given back when the call returns may be written there before
// the call's kernels have run.  An output, which the caller is free to use on the current stream once that has waited for the call, is
// kept from new tensors until such work is done too.
at::Tensor new_on(const at::Tensor &like, at::IntArrayRef shape, at::ScalarType type, PyObject *stream, bool output = true)
{
    const auto options = at::TensorOptions().dtype(type).device(like.device());
    if (stream == Py_None) return at::empty(shape, options);
    const auto handle = (hipStream_t)stream_of(stream);
    const auto current = c10::hip::getCurrentHIPStream(like.device().index());
    if (current.stream() == handle) return at::empty(shape, options);
    struct Restore {
        c10::hip::HIPStream s;
        ~Restore() { c10::hip::setCurrentHIPStream(s); }
    } restore{current};
    c10::hip::setCurrentHIPStream(c10::hip::getStreamFromExternal(handle, like.device().index()));
    at::Tensor t = at::empty(shape, options);
    if (output) t.record_stream(c10::Stream(c10::Stream::UNSAFE, like.device(), current.id()));
    return t;
}

// Memory of the caller's that a call writes `bytes` bytes of `type` to.  The kernels take its address and nothing else, so it is
// looked at here: on the GPU, contiguous and long enough, of that type or, as raw memory, of integers.
const at::Tensor &written(PyObject *o, at::ScalarType type, const char *type_name, int64_t bytes, const char *name)
{
    const at::Tensor &t = tensor(o, name);
    const bool fits = t.scalar_type() == type || c10::isIntegralType(t.scalar_type(), false);
    if (!(t.is_cuda() && fits && t.is_contiguous())) {
        PyErr_Format(PyExc_TypeError, "%s: need a contiguous %s tensor on the GPU", name, type_name);
        throw Failed{};
    }
    if ((int64_t)t.nbytes() < bytes) fail(PyExc_ValueError, "%s: need %lld bytes, got %lld", name, bytes, (long long)t.nbytes());
    return t;
}

// Scratch memory of the caller's: of any type; the library looks at its length, numel() bytes.
const at::Tensor &scratch(PyObject *o, const char *name)
{
    const at::Tensor &t = tensor(o, name);
    if (!(t.is_cuda() && t.is_contiguous())) fail(PyExc_TypeError, "%s: need a contiguous tensor on the GPU", name);
    return t;
}

// Bytes of a matrix; 0 for one so large that the library refuses it.
int64_t bytes_of(int64_t rows, int64_t cols, int64_t each) { return rows <= INT32_MAX && cols <= INT32_MAX ? rows * cols * each : 0; }

// An output: the caller's tensor, or a new one.
struct Out {
    PyObject *given;
    at::Tensor made;
    void *ptr;
    Out(PyObject *o, const at::Tensor &checked) : given(o), ptr(checked.data_ptr()) {}
    explicit Out(at::Tensor t) : given(nullptr), made(std::move(t)), ptr(made.data_ptr()) {}
    PyObject *release()
    {
        if (given) {
            Py_INCREF(given);
            return given;
        }
        return THPVariable_Wrap(std::move(made));
    }
};

Out out_bf16(PyObject *o, const at::Tensor &like, int64_t M, int64_t N, PyObject *stream, const char *name)
{
    if (o != Py_None) return Out(o, written(o, at::kBFloat16, "torch.bfloat16", bytes_of(M, N, 2), name));
    return Out(new_on(like, {M, N}, at::kBFloat16, stream));
}

Out out_f32(PyObject *o, const at::Tensor &like, int64_t rows, PyObject *stream, const char *name)
{
    if (o != Py_None) return Out(o, written(o, at::kFloat, "torch.float32", bytes_of(rows, 1, 4), name));
    return Out(new_on(like, {rows}, at::kFloat, stream));
}

Out out_codes(PyObject *o, const at::Tensor &like, size_t bytes, PyObject *stream, const char *name)
{
    if (o != Py_None) return Out(o, codes(o, bytes, name));
    return Out(new_on(like, {(int64_t)bytes}, at::kByte, stream));
}

// Runs the call without the interpreter lock; an error status goes back as an int for binding.py to raise.
template <class F>
int call(F f)
{
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = f();
    Py_END_ALLOW_THREADS
    return status;
}

// An error inside torch, a failed allocation above all, reaches the caller as it would from torch's own functions: torch's
// exception types and messages, and a Python error that passed through its dispatcher as it was raised.
template <class F>
PyObject *guarded(Py_ssize_t n, Py_ssize_t expected, F f)
{
    HANDLE_TH_ERRORS
    if (n != expected) {
        PyErr_Format(PyExc_TypeError, "need %zd arguments, got %zd", expected, n);
        return nullptr;
    }
    if (!bound) {
        PyErr_SetString(PyExc_RuntimeError, "not bound to a library");
        return nullptr;
    }
    try {
        return f();
    } catch (const Failed &) {
        return nullptr;
    }
    END_HANDLE_TH_ERRORS
}

// (X, Wq, w_scale, group, Y, workspace, bias, stream) -> Y
template <int BITS>
PyObject *forward(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded(n, 8, [&]() -> PyObject * {
        const at::Tensor &X = bf16(a[0], "X"), &ws = f32(a[2], "w_scale");
        int64_t M, K;
        matrix(X, "X", M, K);
        const int64_t N = length(ws, "w_scale");
        const at::Tensor &Wq = codes(a[1], BITS == 4 ? lib.convrot_packed_bytes(N, K) : lib.convrot_packed_bytes8(N, K), "Wq");
        const at::Tensor *workspace = a[5] == Py_None ? nullptr : &scratch(a[5], "workspace");
        Out Y = out_bf16(a[4], X, M, N, a[7], "Y");
        at::Tensor own;
        if (!workspace) {
            const int64_t bytes = BITS == 4 ? lib.convrot_workspace_bytes(M, K) : lib.convrot_workspace_bytes8(M, K);
            own = new_on(X, {std::max<int64_t>(bytes, 256)}, at::kByte, a[7], false);
            workspace = &own;
        }
        const void *bias = bias_of(a[6], N), *x = X.data_ptr(), *w = Wq.data_ptr();
        const float *s = (const float *)ws.data_ptr();
        const int group = (int)integer(a[3]);
        void *stream = stream_of(a[7]), *wp = workspace->data_ptr();
        const size_t wn = workspace->numel();
        const int status = call([&] {
            return BITS == 4 ? lib.convlinear4bit_forward(x, w, s, bias, M, N, K, group, Y.ptr, wp, wn, stream)
                             : lib.convlinear8bit_forward(x, w, s, bias, M, N, K, group, Y.ptr, wp, wn, stream);
        });
        return status ? PyLong_FromLong(status) : Y.release();
    });
}

// (X, Wq, w_scale, group, Y, bias, stream) -> Y
PyObject *forward_noalloc(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded(n, 7, [&]() -> PyObject * {
        const at::Tensor &X = bf16(a[0], "X"), &ws = f32(a[2], "w_scale"), &Y = bf16(a[4], "Y");
        int64_t M, K;
        matrix(X, "X", M, K);
        const int64_t N = length(ws, "w_scale");
        if (Y.dim() != 2 || Y.size(0) != M || Y.size(1) != N) fail(PyExc_ValueError, "%s: need shape [M, N]", "Y");
        const at::Tensor &Wq = codes(a[1], lib.convrot_packed_bytes(N, K), "Wq");
        const void *bias = bias_of(a[5], N), *x = X.data_ptr(), *w = Wq.data_ptr();
        const float *s = (const float *)ws.data_ptr();
        void *y = Y.data_ptr(), *stream = stream_of(a[6]);
        const int group = (int)integer(a[3]);
        const int status = call([&] { return lib.convlinear4bit_forward_noalloc(x, w, s, bias, M, N, K, group, y, stream); });
        if (status) return PyLong_FromLong(status);
        Py_INCREF(a[4]);
        return a[4];
    });
}

// (Xq, x_scale, Wq, w_scale, K, Y, bias, stream) -> Y
template <int BITS>
PyObject *gemm_dequant(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded(n, 8, [&]() -> PyObject * {
        const at::Tensor &xs = f32(a[1], "x_scale"), &ws = f32(a[3], "w_scale");
        const int64_t M = length(xs, "x_scale"), N = length(ws, "w_scale"), K = integer(a[4]);
        auto bytes = BITS == 4 ? lib.convrot_packed_bytes : lib.convrot_packed_bytes8;
        const at::Tensor &Xq = codes(a[0], bytes(M, K), "Xq"), &Wq = codes(a[2], bytes(N, K), "Wq");
        Out Y = out_bf16(a[5], Xq, M, N, a[7], "Y");
        const void *bias = bias_of(a[6], N), *x = Xq.data_ptr(), *w = Wq.data_ptr();
        const float *sx = (const float *)xs.data_ptr(), *sw = (const float *)ws.data_ptr();
        void *stream = stream_of(a[7]);
        const int status = call([&] {
            return (BITS == 4 ? lib.convrot_w4a4_gemm_dequant : lib.convrot_w8a8_gemm_dequant)(x, sx, w, sw, bias, M, N, K, Y.ptr, stream);
        });
        return status ? PyLong_FromLong(status) : Y.release();
    });
}

// (X, group, Xq, x_scale, stream, name of X, name of Xq) -> (Xq, x_scale).  Activations and weights run through the same kernel.
template <int BITS>
PyObject *rotquant(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded(n, 7, [&]() -> PyObject * {
        const char *in_name = PyUnicode_AsUTF8(a[5]), *out_name = PyUnicode_AsUTF8(a[6]);
        if (!in_name || !out_name) throw Failed{};
        const at::Tensor &X = bf16(a[0], in_name);
        int64_t rows, K;
        matrix(X, in_name, rows, K);
        const size_t bytes = BITS == 4 ? lib.convrot_packed_bytes(rows, K) : lib.convrot_packed_bytes8(rows, K);
        Out Xq = out_codes(a[2], X, bytes, a[4], out_name), scale = out_f32(a[3], X, rows, a[4], "scale");
        const void *x = X.data_ptr();
        const int group = (int)integer(a[1]);
        void *stream = stream_of(a[4]);
        const int status = call([&] {
            return (BITS == 4 ? lib.convrot_rotquant_act : lib.convrot_rotquant_act8)(x, rows, K, group, Xq.ptr, (float *)scale.ptr, stream);
        });
        if (status) return PyLong_FromLong(status);
        PyObject *q = Xq.release(), *s = scale.release(), *pair = PyTuple_Pack(2, q, s);
        Py_XDECREF(q);
        Py_XDECREF(s);
        return pair;
    });
}

// (addresses of the entry points named in `names`, in their order)
PyObject *bind(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    Py_ssize_t i = 0;
    Library l;
#define CONVROT_TAKE(name)                                                       \
    if (i >= n || !(l.name = (decltype(l.name))PyLong_AsVoidPtr(a[i++]))) {      \
        if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "no " #name);   \
        return nullptr;                                                          \
    }
    CONVROT_CALLS(CONVROT_TAKE)
#undef CONVROT_TAKE
    lib = l;
    bound = true;
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"bind", (PyCFunction)(void (*)(void))bind, METH_FASTCALL, nullptr},
    {"forward4", (PyCFunction)(void (*)(void))forward<4>, METH_FASTCALL, nullptr},
    {"forward8", (PyCFunction)(void (*)(void))forward<8>, METH_FASTCALL, nullptr},
    {"forward4_noalloc", (PyCFunction)(void (*)(void))forward_noalloc, METH_FASTCALL, nullptr},
    {"gemm_dequant4", (PyCFunction)(void (*)(void))gemm_dequant<4>, METH_FASTCALL, nullptr},
    {"gemm_dequant8", (PyCFunction)(void (*)(void))gemm_dequant<8>, METH_FASTCALL, nullptr},
    {"rotquant4", (PyCFunction)(void (*)(void))rotquant<4>, METH_FASTCALL, nullptr},
    {"rotquant8", (PyCFunction)(void (*)(void))rotquant<8>, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_torch_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__torch_calls()
{
    PyObject *m = PyModule_Create(&module);
#define CONVROT_NAME(name) #name " "
    if (m && PyModule_AddStringConstant(m, "names", CONVROT_CALLS(CONVROT_NAME)) < 0) Py_CLEAR(m);
#undef CONVROT_NAME
    return m;
}
