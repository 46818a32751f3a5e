// Argument marshalling of the per-token calls in native code: torch tensors in, the C ABI of include/smoothrot.h called
// on the current stream, tensors out.  No computation here.
//
// Why: a decode step's kernels run 5 - 10 us each, and marshalling through Python and ctypes cost 8.5 - 15 us per call
// (3 us of it torch.cuda.current_stream(), 1.7 us per torch.empty, 5.4 us for the fill kernel of a zeroed tile buffer),
// so the host, not the GPU, set the pace of everything below about 300 tokens.  Here a call costs the launch
// (~3.8 us per kernel) and about a microsecond.
//
// Every function takes positional arguments (binding.py has the signatures and their defaults) and returns its
// outputs, or the status as an int where the library refused the call.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/hip/EmptyTensor.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/smoothrot.h"

#include <exception>

namespace {

struct Raised {};                                        // a Python exception is set

[[noreturn]] void value_error(const char *format, const char *a, const char *b = "")
{
    PyErr_Format(PyExc_ValueError, format, a, b);
    throw Raised();
}

const at::Tensor &tensor(PyObject *o, const char *name)
{
    if (!THPVariable_Check(o)) {
        PyErr_Format(PyExc_TypeError, "%s must be a tensor", name);
        throw Raised();
    }
    return THPVariable_Unpack(o);
}

// a device tensor of the given type, contiguous along its last dimension
const at::Tensor &device_tensor(PyObject *o, at::ScalarType type, const char *name)
{
    const at::Tensor &t = tensor(o, name);
    if (!t.is_cuda()) value_error("%s must be a device tensor", name);
    if (t.scalar_type() != type) value_error("%s must have dtype torch.%s", name, type == at::kHalf ? "float16" : type == at::kByte ? "uint8" : "float32");
    if ((t.dim() == 2 && t.stride(1) != 1) || (t.dim() == 1 && t.numel() > 1 && t.stride(0) != 1))
        value_error("%s must be contiguous along its last dimension", name);
    return t;
}
const at::Tensor &matrix(PyObject *o, at::ScalarType type, const char *name)
{
    const at::Tensor &t = device_tensor(o, type, name);
    if (t.dim() != 2) value_error("%s must have two dimensions", name);
    return t;
}

// Addresses are taken before the lock is released: data_ptr() throws for a tensor without memory of its own (inside vmap, ..).
void *pointer(PyObject *o, const char *name) { return o == Py_None ? nullptr : tensor(o, name).data_ptr(); }
float *floats(PyObject *o, const char *name) { return static_cast<float *>(pointer(o, name)); }
float *floats(const at::Tensor &t) { return static_cast<float *>(t.data_ptr()); }
uint8_t *bytes(const at::Tensor &t) { return static_cast<uint8_t *>(t.data_ptr()); }
int64_t integer(PyObject *o)
{
    const int64_t v = PyLong_AsLongLong(o);
    if (v == -1 && PyErr_Occurred()) throw Raised();
    return v;
}
float real(PyObject *o)
{
    const double v = PyFloat_AsDouble(o);
    if (v == -1.0 && PyErr_Occurred()) throw Raised();
    return (float)v;
}
bool truth(PyObject *o)
{
    const int v = PyObject_IsTrue(o);
    if (v < 0) throw Raised();
    return v != 0;
}
int64_t row_stride(const at::Tensor &t) { return t.size(0) > 1 ? t.stride(0) : t.size(1); }

at::Tensor empty(at::IntArrayRef shape, at::ScalarType type, const at::Tensor &like)
{
    return at::detail::empty_cuda(shape, type, like.device(), std::nullopt);
}
// the caller's tensor, or a new one
at::Tensor output(PyObject *o, const char *name, at::IntArrayRef shape, at::ScalarType type, const at::Tensor &like)
{
    return o == Py_None ? empty(shape, type, like) : tensor(o, name);
}
void *stream() { return c10::hip::getCurrentHIPStream().stream(); }

PyObject *pair(const at::Tensor &a, const at::Tensor &b) { return Py_BuildValue("(NN)", THPVariable_Wrap(a), THPVariable_Wrap(b)); }

// calls into the library without holding the interpreter's lock (the library does not throw)
template <typename F> int released(F f)
{
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = f();
    Py_END_ALLOW_THREADS
    return status;
}

template <PyObject *(*F)(PyObject *const *), int N> PyObject *entry(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    if (n != N) {
        PyErr_Format(PyExc_TypeError, "%d arguments expected, %zd given", N, n);
        return nullptr;
    }
    try {
        return F(args);
    } catch (const Raised &) {
    } catch (...) {                                      // as torch raises them: out of memory, bad index, ..
        torch::translate_exception_to_python(std::current_exception());
    }
    return nullptr;
}

// X, inv_s, clip, Xq, x_scale
PyObject *fwht_quant_act(PyObject *const *a)
{
    const at::Tensor &X = matrix(a[0], at::kHalf, "X");
    const int64_t M = X.size(0), K = X.size(1);
    const at::Tensor Xq = output(a[3], "Xq", {M, K / 2}, at::kByte, X), xs = output(a[4], "x_scale", {M}, at::kFloat, X);
    const float clip = real(a[2]);
    const float *inv = floats(a[1], "inv_s");
    const void *x = X.data_ptr();
    uint8_t *q = bytes(Xq);
    float *scale = floats(xs);
    const int64_t ldx = row_stride(X);
    void *st = stream();
    const int status = released([&] { return sr_fwht_quant_act(x, M, K, ldx, inv, clip, q, scale, st); });
    return status ? PyLong_FromLong(status) : pair(Xq, xs);
}

// X, n_heads, across, inv_s, clip, Xq, x_scale
PyObject *fwht_quant_act_heads(PyObject *const *a)
{
    const at::Tensor &X = matrix(a[0], at::kHalf, "X");
    const int64_t M = X.size(0), K = X.size(1), heads = integer(a[1]);
    const int across = truth(a[2]);
    const at::Tensor Xq = output(a[5], "Xq", {M, K / 2}, at::kByte, X), xs = output(a[6], "x_scale", {M}, at::kFloat, X);
    const float clip = real(a[4]);
    const float *inv = floats(a[3], "inv_s");
    const void *x = X.data_ptr();
    uint8_t *q = bytes(Xq);
    float *scale = floats(xs);
    const int64_t ldx = row_stride(X);
    void *st = stream();
    const int status = released([&] { return sr_fwht_quant_act_heads(x, M, K, ldx, heads, across, inv, clip, q, scale, st); });
    return status ? PyLong_FromLong(status) : pair(Xq, xs);
}

// a buffer whose bytes the library may read as the next operand: (address, bytes)
void warm_region(PyObject *o, const void *&p, size_t &size)
{
    p = nullptr;
    size = 0;
    if (o == Py_None) return;
    const at::Tensor &t = tensor(o, "warm");
    if (!t.is_cuda() || !t.is_contiguous()) value_error("%s must be a contiguous device tensor", "warm");
    p = t.data_ptr();
    size = t.nbytes();
}

int64_t tile_bytes(int64_t M, int64_t K)
{
    const size_t n = sr_f6_tiles_bytes(M, K);
    return n > 16 ? (int64_t)n : 16;
}

// X, inv_s, clip, X6, x_scale, warm
PyObject *fwht_quant_act_f6(PyObject *const *a)
{
    const at::Tensor &X = matrix(a[0], at::kHalf, "X");
    const int64_t M = X.size(0), K = X.size(1);
    const at::Tensor X6 = output(a[3], "X6", {tile_bytes(M, K)}, at::kByte, X), xs = output(a[4], "x_scale", {M}, at::kFloat, X);
    const float clip = real(a[2]);
    const float *inv = floats(a[1], "inv_s");
    const void *warm;
    size_t warm_bytes;
    warm_region(a[5], warm, warm_bytes);
    const void *x = X.data_ptr();
    uint8_t *q = bytes(X6);
    float *scale = floats(xs);
    const int64_t ldx = row_stride(X);
    void *st = stream();
    const int status = released([&] { return sr_fwht_quant_act_f6_warm(x, M, K, ldx, inv, clip, q, scale, warm, warm_bytes, st); });
    return status ? PyLong_FromLong(status) : pair(X6, xs);
}

// G, U, inv_s, clip, Xq or X6, x_scale, tiles
PyObject *swiglu_fwht_quant_act(PyObject *const *a)
{
    const at::Tensor &G = matrix(a[0], at::kHalf, "G"), &U = matrix(a[1], at::kHalf, "U");
    const int64_t M = U.size(0), K = U.size(1);
    if (G.size(0) != M || G.size(1) != K) value_error("%s must have the same shape", "G and U");
    const bool tiles = truth(a[6]);
    const at::Tensor Q = tiles ? output(a[4], "X6", {tile_bytes(M, K)}, at::kByte, U) : output(a[4], "Xq", {M, K / 2}, at::kByte, U);
    const at::Tensor xs = output(a[5], "x_scale", {M}, at::kFloat, U);
    const float clip = real(a[3]);
    const float *inv = floats(a[2], "inv_s");
    const void *g = G.data_ptr(), *u = U.data_ptr();
    uint8_t *q = bytes(Q);
    float *scale = floats(xs);
    const int64_t ldg = row_stride(G), ldu = row_stride(U);
    void *st = stream();
    const auto f = tiles ? sr_swiglu_fwht_quant_act_f6 : sr_swiglu_fwht_quant_act;
    const int status = released([&] { return f(g, u, M, K, ldg, ldu, inv, clip, q, scale, st); });
    return status ? PyLong_FromLong(status) : pair(Q, xs);
}

// Xq, x_scale, Wq, w_scale, out_dtype, Y, workspace
PyObject *w4a4_gemm(PyObject *const *a)
{
    const at::Tensor &Xq = matrix(a[0], at::kByte, "Xq"), &Wq = matrix(a[2], at::kByte, "Wq");
    const int64_t M = Xq.size(0), Kb = Xq.size(1), N = Wq.size(0);
    if (Wq.size(1) != Kb) value_error("%s disagree on K", "Xq and Wq");
    const int type = (int)integer(a[4]);
    const at::Tensor Y = output(a[5], "Y", {M, N}, type == SR_F16 ? at::kHalf : at::kInt, Xq);
    const float *xs = floats(a[1], "x_scale"), *ws = floats(a[3], "w_scale");
    at::Tensor work;
    if (a[6] != Py_None) work = tensor(a[6], "workspace");
    else if (const size_t need = sr_gemm_workspace_bytes(M, N, 2 * Kb)) work = empty({(int64_t)need}, at::kByte, Xq);
    const int64_t ldy = M > 1 ? Y.stride(0) : N;
    const uint8_t *x = bytes(Xq), *w = bytes(Wq);
    void *y = Y.data_ptr(), *scratch = work.defined() ? work.data_ptr() : nullptr, *st = stream();
    const size_t scratch_bytes = work.defined() ? (size_t)work.numel() : 0;
    const int status = released([&] { return sr_w4a4_gemm(x, xs, w, ws, M, N, 2 * Kb, y, ldy, type, scratch, scratch_bytes, st); });
    return status ? PyLong_FromLong(status) : THPVariable_Wrap(Y);
}

// X6, x_scale, W6, w_scale, M, N, K, out_dtype, Y, warm
PyObject *w4a4_gemm_f6(PyObject *const *a)
{
    const at::Tensor &X6 = device_tensor(a[0], at::kByte, "X6"), &W6 = device_tensor(a[2], at::kByte, "W6");
    const int64_t M = integer(a[4]), N = integer(a[5]), K = integer(a[6]);
    if ((size_t)X6.numel() < sr_f6_tiles_bytes(M, K) || (size_t)W6.numel() < sr_f6_tiles_bytes(N, K))
        value_error("%s are smaller than sr_f6_tiles_bytes says", "tile buffers");
    const int type = (int)integer(a[7]);
    const at::Tensor Y = output(a[8], "Y", {M, N}, type == SR_F16 ? at::kHalf : at::kInt, X6);
    const float *xs = floats(a[1], "x_scale"), *ws = floats(a[3], "w_scale");
    const void *warm;
    size_t warm_bytes;
    warm_region(a[9], warm, warm_bytes);
    const int64_t ldy = M > 1 ? Y.stride(0) : N;
    const uint8_t *x = bytes(X6), *w = bytes(W6);
    void *y = Y.data_ptr(), *st = stream();
    const int status = released([&] { return sr_w4a4_gemm_f6_warm(x, xs, w, ws, M, N, K, y, ldy, type, warm, warm_bytes, nullptr, 0, st); });
    return status ? PyLong_FromLong(status) : THPVariable_Wrap(Y);
}

// X, inv_s, Wq, w_scale, clip, Y, Xq_out, x_scale_out, workspace
PyObject *w4a4_linear_decode(PyObject *const *a)
{
    const at::Tensor &X = matrix(a[0], at::kHalf, "X"), &Wq = matrix(a[2], at::kByte, "Wq");
    const int64_t M = X.size(0), K = X.size(1), N = Wq.size(0);
    if (Wq.size(1) * 2 != K) value_error("%s disagree on K", "X and Wq");
    const at::Tensor Y = output(a[5], "Y", {M, N}, at::kHalf, X);
    const float *inv = floats(a[1], "inv_s"), *ws = floats(a[3], "w_scale");
    uint8_t *xq = static_cast<uint8_t *>(pointer(a[6], "Xq_out"));
    float *xs = floats(a[7], "x_scale_out");
    const float clip = real(a[4]);
    at::Tensor work;
    if (a[8] != Py_None) work = tensor(a[8], "workspace");
    else if (const size_t need = sr_linear_decode_workspace_bytes(M, K)) work = empty({(int64_t)need}, at::kByte, X);
    const int64_t ldx = row_stride(X), ldy = M > 1 ? Y.stride(0) : N;
    const void *x = X.data_ptr();
    const uint8_t *w = bytes(Wq);
    void *y = Y.data_ptr(), *scratch = work.defined() ? work.data_ptr() : nullptr, *st = stream();
    const size_t scratch_bytes = work.defined() ? (size_t)work.numel() : 0;
    const int status = released([&] {
        return sr_w4a4_linear_decode(x, M, K, ldx, inv, clip, w, ws, N, y, ldy, xq, xs, scratch, scratch_bytes, st);
    });
    return status ? PyLong_FromLong(status) : THPVariable_Wrap(Y);
}

// X, group, clip, Q, scale, zero
PyObject *kv_quant_asym(PyObject *const *a)
{
    const at::Tensor &X = matrix(a[0], at::kHalf, "X");
    const int64_t rows = X.size(0), D = X.size(1), group = integer(a[1]);
    if (group <= 0) return PyLong_FromLong(SR_ERR_ARG);
    const int64_t groups = D / group > 1 ? D / group : 1;
    const at::Tensor Q = output(a[3], "Q", {rows, D / 2}, at::kByte, X), scale = output(a[4], "scale", {rows, groups}, at::kFloat, X),
                     zero = output(a[5], "zero", {rows, groups}, at::kFloat, X);
    const float clip = real(a[2]);
    const void *x = X.data_ptr();
    uint8_t *q = bytes(Q);
    float *scales = floats(scale), *zeros = floats(zero);
    const int64_t ldx = row_stride(X);
    void *st = stream();
    const int status = released([&] { return sr_kv_quant_asym(x, rows, D, ldx, group, clip, q, scales, zeros, st); });
    return status ? PyLong_FromLong(status)
                  : Py_BuildValue("(NNN)", THPVariable_Wrap(Q), THPVariable_Wrap(scale), THPVariable_Wrap(zero));
}

PyObject *current_stream(PyObject *const *) { return PyLong_FromVoidPtr(stream()); }

#define SR_ENTRY(F, N) {#F, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(entry<F, N>)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {SR_ENTRY(fwht_quant_act, 5), SR_ENTRY(fwht_quant_act_heads, 7), SR_ENTRY(fwht_quant_act_f6, 6),
                         SR_ENTRY(swiglu_fwht_quant_act, 7), SR_ENTRY(w4a4_gemm, 7), SR_ENTRY(w4a4_gemm_f6, 10),
                         SR_ENTRY(w4a4_linear_decode, 9), SR_ENTRY(kv_quant_asym, 6), SR_ENTRY(current_stream, 0), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal(void)
{
    PyObject *m = PyModule_Create(&module_def);
    if (m && PyModule_AddStringConstant(m, "torch_version", SR_TORCH_VERSION) < 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
