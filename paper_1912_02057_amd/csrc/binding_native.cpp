// The hot calls of the Python binding in native code: argument checks, marshalling and the call into
// librtn for one entry point each.  A pass over a network's layers at batch 1 is bound by the host, and
// the same work through ctypes took 6 to 10 us per call (it takes about 1 us here); the GPU needs 4 to
// 8 us for such a layer.  binding.py keeps the public signatures, allocates default outputs and
// raises on a status; the checks below raise what it raised: AssertionError for a tensor of the
// wrong device, type or layout, ValueError for a code tensor that does not hold the stated codes.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/core/TensorBase.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/rtn.h"

namespace {

// Thrown after a Python error has been set.
struct PyError {};

[[noreturn]] void fail(PyObject* type, const char* fmt, const char* what)
{
    PyErr_Format(type, fmt, what);
    throw PyError();
}

int64_t integer(PyObject* o)
{
    const long long v = PyLong_AsLongLong(o);
    if (v == -1 && PyErr_Occurred()) throw PyError();
    return v;
}
int truth(PyObject* o)
{
    const int v = PyObject_IsTrue(o);
    if (v < 0) throw PyError();
    return v;
}

const at::Tensor& tensor(PyObject* o, const char* what)
{
    if (!THPVariable_Check(o)) fail(PyExc_TypeError, "%s: a torch tensor is required", what);
    return THPVariable_Unpack(o);
}

// Data pointer of a contiguous device tensor of the given type; None -> NULL.
void* dev(PyObject* o, c10::ScalarType type, const char* what, bool nullable = true)
{
    if (nullable && o == Py_None) return nullptr;
    const at::Tensor& t = tensor(o, what);
    if (!t.is_cuda() || t.scalar_type() != type || !t.is_contiguous())
        fail(PyExc_AssertionError, "%s: a contiguous device tensor of the documented type is required", what);
    return t.data_ptr();
}
// Any tensor's storage, unchecked (workspaces, prepared weights).
void* raw(PyObject* o, const char* what) { return o == Py_None ? nullptr : tensor(o, what).data_ptr(); }
size_t raw_bytes(PyObject* o, const char* what) { return o == Py_None ? 0 : tensor(o, what).nbytes(); }

// The library takes raw pointers: make sure the tensor really holds `rows` rows of K codes in format
// fmt, so that a tensor packed in another format cannot be read out of bounds.
void* codes(PyObject* o, int64_t rows, int64_t K, rtn_code_format fmt, const char* what)
{
    const at::Tensor& t = tensor(o, what);
    const size_t need = rtn_codes_bytes(fmt, rows, K), have = t.nbytes();
    if (!(t.is_cuda() && t.is_contiguous() && have >= need)) {
        PyErr_Format(PyExc_ValueError, "%s: %zu bytes, but %lld rows of %lld codes in format %d need %zu", what, have,
                     (long long)rows, (long long)K, (int)fmt, need);
        throw PyError();
    }
    const c10::ScalarType type = t.scalar_type();
    if ((fmt == RTN_CODE_FP4 && type != c10::kByte) || (fmt == RTN_CODE_I8 && type != c10::kChar) ||
        (fmt == RTN_CODE_BITPLANE && type != c10::kLong && type != c10::kUInt64))
        fail(PyExc_ValueError, "%s: dtype does not match the code format", what);
    return t.data_ptr();
}

// A python number (host scalar) or a device float32 vector.
struct Gran {
    float s = 0.0f;
    const float* ptr = nullptr;
    rtn_gran gran = RTN_SCALAR;
    Gran(PyObject* o, const char* what)
    {
        if (o == Py_None) return;
        if (THPVariable_Check(o)) {
            ptr = (const float*)dev(o, c10::kFloat, what, false);
            gran = RTN_VECTOR;
        } else {
            const double v = PyFloat_AsDouble(o);
            if (v == -1.0 && PyErr_Occurred()) throw PyError();
            s = (float)v;
            ptr = &s;
        }
    }
    Gran(const Gran&) = delete;
};

const rtn_epilogue* epilogue(PyObject* o)  // address of an Epilogue's struct, or None
{
    if (o == Py_None) return nullptr;
    const void* p = PyLong_AsVoidPtr(o);
    if (!p && PyErr_Occurred()) throw PyError();
    return (const rtn_epilogue*)p;
}

// torch's current stream.  On a host without a GPU the library's own checks must be what raises.
void* stream()
{
    try {
        return (void*)c10::hip::getCurrentHIPStream().stream();
    } catch (const c10::Error&) {
        if (c10::hip::device_count() > 0) throw;
        return nullptr;
    }
}

// The interpreter's lock is given up around a call into the library, as ctypes gives it up: a launch that
// loads its code object or waits for room in the queue must not stop every other Python thread.  The
// arguments are converted before (the caller's frame keeps them alive meanwhile).
struct Unlocked {
    PyThreadState* state = PyEval_SaveThread();
    ~Unlocked() { PyEval_RestoreThread(state); }
};

// Runs `f` on the arguments; a C++ exception or a wrong argument count becomes a Python error.
template <class F>
PyObject* call(Py_ssize_t want, Py_ssize_t n, F f)
{
    if (n != want) {
        PyErr_Format(PyExc_TypeError, "%zd arguments expected, got %zd", want, n);
        return nullptr;
    }
    try {
        return PyLong_FromLong(f());
    } catch (const PyError&) {
        return nullptr;
    } catch (const std::exception& e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
}
typedef PyObject* const* Args;

// x, layout, d0, d1, d2, d3, lo, hi, fmt, codes, sum_t
PyObject* pack(PyObject*, Args a, Py_ssize_t n)
{
    return call(11, n, [&] {
        const Gran lo(a[6], "lo"), hi(a[7], "hi");
        if (lo.gran != hi.gran) fail(PyExc_AssertionError, "%s: lo and hi must both be scalars or both vectors", "ternarize_pack");
        const float* x = (const float*)dev(a[0], c10::kFloat, "x");
        const rtn_layout layout = (rtn_layout)integer(a[1]);
        const int64_t d0 = integer(a[2]), d1 = integer(a[3]), d2 = integer(a[4]), d3 = integer(a[5]);
        const rtn_code_format fmt = (rtn_code_format)integer(a[8]);
        void* out = raw(a[9], "codes");
        int32_t* sum = (int32_t*)dev(a[10], c10::kInt, "sum_t");
        void* st = stream();
        const Unlocked u;
        return rtn_ternarize_pack(x, layout, d0, d1, d2, d3, lo.ptr, hi.ptr, lo.gran, fmt, out, sum, st);
    });
}

// fmt, path, a_codes, w_codes, M, N, K, acc_out, ep, y_out
PyObject* gemm(PyObject*, Args a, Py_ssize_t n)
{
    return call(10, n, [&] {
        const rtn_code_format fmt = (rtn_code_format)integer(a[0]);
        const rtn_path path = (rtn_path)integer(a[1]);
        const int64_t M = integer(a[4]), N = integer(a[5]), K = integer(a[6]);
        const void *ac = codes(a[2], M, K, fmt, "a_codes"), *wc = codes(a[3], N, K, fmt, "w_codes");
        int32_t* acc = (int32_t*)dev(a[7], c10::kInt, "acc_out");
        const rtn_epilogue* ep = epilogue(a[8]);
        float* y = (float*)dev(a[9], c10::kFloat, "y_out");
        void* st = stream();
        const Unlocked u;
        return rtn_ternary_gemm(fmt, path, ac, wc, M, N, K, acc, ep, y, nullptr, 0, st);
    });
}

// fmt, path, a_codes, w_codes, Nb, C, H, W, O, KH, KW, stride, pad, pad_mode, acc_out, ep, y_out, workspace
PyObject* conv2d(PyObject*, Args a, Py_ssize_t n)
{
    return call(18, n, [&] {
        const rtn_code_format fmt = (rtn_code_format)integer(a[0]);
        const rtn_path path = (rtn_path)integer(a[1]);
        const int64_t Nb = integer(a[4]), C = integer(a[5]), H = integer(a[6]), W = integer(a[7]), O = integer(a[8]);
        const int KH = (int)integer(a[9]), KW = (int)integer(a[10]), stride = (int)integer(a[11]), pad = (int)integer(a[12]);
        const rtn_pad_mode mode = (rtn_pad_mode)integer(a[13]);
        const void* ac = codes(a[2], Nb * H * W, C, fmt, "a_codes");
        const void* wc = codes(a[3], O * KH * KW, C, fmt, "w_codes");
        int32_t* acc = (int32_t*)dev(a[14], c10::kInt, "acc_out");
        const rtn_epilogue* ep = epilogue(a[15]);
        float* y = (float*)dev(a[16], c10::kFloat, "y_out");
        void* ws = raw(a[17], "workspace");
        const size_t wsb = raw_bytes(a[17], "workspace");
        void* st = stream();
        const Unlocked u;
        return rtn_ternary_conv2d_implicit_gemm(fmt, path, ac, wc, Nb, C, H, W, O, KH, KW, stride, pad, mode, acc, ep, y, ws, wsb, st);
    });
}

// fmt, path, a_codes, w_codes, Nb, C, H, W, O, KH, KW, stride, pad, pad_mode, ep, residual, relu_out, lo, hi, y_out, codes_out,
// workspace
PyObject* conv2d_ternarize(PyObject*, Args a, Py_ssize_t n)
{
    return call(22, n, [&] {
        const rtn_code_format fmt = (rtn_code_format)integer(a[0]);
        const rtn_path path = (rtn_path)integer(a[1]);
        const int64_t Nb = integer(a[4]), C = integer(a[5]), H = integer(a[6]), W = integer(a[7]), O = integer(a[8]);
        const int KH = (int)integer(a[9]), KW = (int)integer(a[10]), stride = (int)integer(a[11]), pad = (int)integer(a[12]);
        const rtn_pad_mode mode = (rtn_pad_mode)integer(a[13]);
        const void* ac = codes(a[2], Nb * H * W, C, fmt, "a_codes");
        const void* wc = codes(a[3], O * KH * KW, C, fmt, "w_codes");
        const int64_t OH = stride > 0 ? (H + 2 * pad - KH) / stride + 1 : 0, OW = stride > 0 ? (W + 2 * pad - KW) / stride + 1 : 0;
        void* co = codes(a[20], Nb * OH * OW, O, fmt, "codes_out");
        const Gran lo(a[17], "lo"), hi(a[18], "hi");
        if (lo.gran != hi.gran) fail(PyExc_AssertionError, "%s: lo and hi must both be scalars or both vectors", "ternary_conv2d_ternarize");
        const rtn_epilogue* ep = epilogue(a[14]);
        const float* res = (const float*)dev(a[15], c10::kFloat, "residual");
        const int relu_out = truth(a[16]);
        float* y = (float*)dev(a[19], c10::kFloat, "y_out");
        void* ws = raw(a[21], "workspace");
        const size_t wsb = raw_bytes(a[21], "workspace");
        void* st = stream();
        const Unlocked u;
        return rtn_ternary_conv2d_ternarize(fmt, path, ac, wc, Nb, C, H, W, O, KH, KW, stride, pad, mode, ep, res, relu_out, lo.ptr, hi.ptr,
                                            lo.gran, y, co, ws, wsb, st);
    });
}

// a_codes, w_codes, Nb, C, H, W, KH, KW, stride, pad, pad_mode, acc_out, ep, y_out
PyObject* depthwise(PyObject*, Args a, Py_ssize_t n)
{
    return call(14, n, [&] {
        const int64_t Nb = integer(a[2]), C = integer(a[3]), H = integer(a[4]), W = integer(a[5]);
        const int KH = (int)integer(a[6]), KW = (int)integer(a[7]), stride = (int)integer(a[8]), pad = (int)integer(a[9]);
        const rtn_pad_mode mode = (rtn_pad_mode)integer(a[10]);
        const void* ac = codes(a[0], Nb * H * W, C, RTN_CODE_I8, "a_codes");
        const void* wc = codes(a[1], C, KH * KW, RTN_CODE_I8, "w_codes");
        int32_t* acc = (int32_t*)dev(a[11], c10::kInt, "acc_out");
        const rtn_epilogue* ep = epilogue(a[12]);
        float* y = (float*)dev(a[13], c10::kFloat, "y_out");
        void* st = stream();
        const Unlocked u;
        return rtn_ternary_depthwise_conv2d(ac, wc, Nb, C, H, W, KH, KW, stride, pad, mode, acc, ep, y, st);
    });
}

// x, w_codes or prepared, is_prepared, M, N, K, alpha_w, relu, bn_scale, bn_shift, y_out, workspace
PyObject* weight_gemm(PyObject*, Args a, Py_ssize_t n)
{
    return call(12, n, [&] {
        const Gran al(a[6], "alpha_w");
        auto fn = truth(a[2]) ? rtn_ternary_weight_gemm_prepared : rtn_ternary_weight_gemm;
        const float* x = (const float*)dev(a[0], c10::kFloat, "x");
        const void* w = raw(a[1], "w_codes");
        const int64_t M = integer(a[3]), N = integer(a[4]), K = integer(a[5]);
        const int relu = truth(a[7]);
        const float *bs = (const float*)dev(a[8], c10::kFloat, "bn_scale"), *bh = (const float*)dev(a[9], c10::kFloat, "bn_shift");
        float* y = (float*)dev(a[10], c10::kFloat, "y_out");
        void* ws = raw(a[11], "workspace");
        const size_t wsb = raw_bytes(a[11], "workspace");
        void* st = stream();
        const Unlocked u;
        return fn(x, w, M, N, K, al.ptr, al.gran, relu, bs, bh, y, ws, wsb, st);
    });
}

// x, prepared, Nb, C, H, W, O, KH, KW, stride, pad, relu, y_out, workspace
PyObject* weight_conv2d_prepared(PyObject*, Args a, Py_ssize_t n)
{
    return call(14, n, [&] {
        const float* x = (const float*)dev(a[0], c10::kFloat, "x");
        const void* w = raw(a[1], "prepared");
        const int64_t Nb = integer(a[2]), C = integer(a[3]), H = integer(a[4]), W = integer(a[5]), O = integer(a[6]);
        const int KH = (int)integer(a[7]), KW = (int)integer(a[8]), stride = (int)integer(a[9]), pad = (int)integer(a[10]);
        const int relu = truth(a[11]);
        float* y = (float*)dev(a[12], c10::kFloat, "y_out");
        void* ws = raw(a[13], "workspace");
        const size_t wsb = raw_bytes(a[13], "workspace");
        void* st = stream();
        const Unlocked u;
        return rtn_ternary_weight_conv2d_prepared(x, w, Nb, C, H, W, O, KH, KW, stride, pad, relu, y, ws, wsb, st);
    });
}

// a, grad_out, n, lo, hi, gamma, grad_in, sums, workspace
PyObject* activation_backward(PyObject*, Args a, Py_ssize_t n)
{
    return call(9, n, [&] {
        const Gran lo(a[3], "lo"), hi(a[4], "hi"), ga(a[5], "gamma");
        const float *x = (const float*)dev(a[0], c10::kFloat, "a"), *g = (const float*)dev(a[1], c10::kFloat, "grad_out");
        const int64_t count = integer(a[2]);
        float* gi = (float*)dev(a[6], c10::kFloat, "grad_in");
        double* sums = (double*)dev(a[7], c10::kDouble, "sums");
        void* ws = raw(a[8], "workspace");
        const size_t wsb = raw_bytes(a[8], "workspace");
        void* st = stream();
        const Unlocked u;
        return rtn_activation_backward(x, g, count, lo.ptr, hi.ptr, ga.ptr, gi, sums, ws, wsb, st);
    });
}

// w, grad_out, O, K, lo, hi, k_w, b_w, alpha, grad_w, sums
PyObject* weight_backward(PyObject*, Args a, Py_ssize_t n)
{
    return call(11, n, [&] {
        const Gran lo(a[4], "lo"), hi(a[5], "hi");
        const float *w = (const float*)dev(a[0], c10::kFloat, "w"), *g = (const float*)dev(a[1], c10::kFloat, "grad_out");
        const int64_t O = integer(a[2]), K = integer(a[3]);
        const float *kw = (const float*)dev(a[6], c10::kFloat, "k_w"), *bw = (const float*)dev(a[7], c10::kFloat, "b_w"),
                    *al = (const float*)dev(a[8], c10::kFloat, "alpha");
        float* gw = (float*)dev(a[9], c10::kFloat, "grad_w");
        double* sums = (double*)dev(a[10], c10::kDouble, "sums");
        void* st = stream();
        const Unlocked u;
        return rtn_weight_backward(w, g, O, K, lo.ptr, hi.ptr, kw, bw, al, gw, sums, st);
    });
}

#define FAST(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {FAST(pack), FAST(gemm), FAST(conv2d), FAST(conv2d_ternarize), FAST(depthwise), FAST(weight_gemm),
                         FAST(weight_conv2d_prepared), FAST(activation_backward), FAST(weight_backward), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) { return PyModule_Create(&module); }
