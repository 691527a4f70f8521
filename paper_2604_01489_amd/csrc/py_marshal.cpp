// Argument marshalling of the binding's calls in native code (binding.py): the checks and conversions that binding.py spells out, for the arguments
// that programs pass -- exact ints, floats, strings and torch tensors on the device -- and the call itself, without the GIL.  Anything else (another
// type, a tensor subclass, a value out of range, a tensor on the CPU or too small for the sizes) returns None, and binding.py's own
// code takes the call and raises what it always has.  Nothing is kept between calls; the entry point's address comes with each.
//
// What it saves, host time a call: an fp32 product 7.0 -> 4.0 us, the widened operator 9.7 -> 5.1, a convolution 7.5 -> 4.2, the two calls of a row sum 15.0 ->
// 10.5; 4 us of each launch are the library and the runtime.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <climits>
#include <cmath>
#include <torch/csrc/autograd/python_variable.h>
#include <ATen/PythonTorchFunctionTLS.h>

#include "../../include/gemm_epilogue.h"
#include "py_call.h"

namespace {

using ge_py::Decline;
using ge_py::without_gil;

int to_int(PyObject *o)
{
    if (!PyLong_CheckExact(o)) throw Decline{};
    int overflow = 0;
    const long v = PyLong_AsLongAndOverflow(o, &overflow);
    if (overflow || v < INT_MIN || v > INT_MAX) throw Decline{};
    return (int)v;
}

int to_flag(PyObject *o)
{
    if (o == Py_True) return 1;
    if (o == Py_False) return 0;
    return to_int(o) ? 1 : 0;
}

float to_float(PyObject *o)
{
    if (PyFloat_CheckExact(o)) return (float)PyFloat_AS_DOUBLE(o);
    return (float)to_int(o);
}

void *to_address(PyObject *o)
{
    void *p = PyLong_CheckExact(o) ? PyLong_AsVoidPtr(o) : nullptr;
    if (!p) { PyErr_Clear(); throw Decline{}; }
    return p;
}

int one_of(PyObject *o, const char *const *names, int n)
{
    if (!PyUnicode_CheckExact(o)) throw Decline{};
    for (int i = 0; i < n; ++i)
        if (PyUnicode_CompareWithASCIIString(o, names[i]) == 0) return i;
    throw Decline{};
}

int to_act(PyObject *o)
{
    static const char *const names[] = {"none", "relu", "gelu_tanh"};
    return one_of(o, names, 3);
}

int to_plan(PyObject *o)
{
    static const char *const names[] = {"auto", "direct", "splitk"};
    return one_of(o, names, 3);
}

int to_structure(PyObject *o)
{
    static const char *const names[] = {"general", "lower", "upper", "sym_lower", "sym_upper"};
    return one_of(o, names, 5);
}

// a device tensor, or (where one may be missing) null for None
const at::Tensor *to_tensor(PyObject *o, bool optional = false)
{
    if (optional && o == Py_None) return nullptr;
    if (!THPVariable_CheckExact(o)) throw Decline{};
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.is_cuda()) throw Decline{};
    return &t;
}

void *address(const at::Tensor *t) { return t ? t->data_ptr() : nullptr; }
int kind(const at::Tensor *t) { return t->scalar_type() == at::kFloat ? GE_DTYPE_F32 : GE_DTYPE_BF16; }

// binding.py's _require_extent
void extent(const at::Tensor *t, long long rows, long long cols, long long ld, long long batch)
{
    if (!t || rows < 1 || cols < 1 || batch < 1 || ld < cols) return;
    if ((__int128)t->numel() < ((__int128)batch * rows - 1) * ld + cols) throw Decline{};
}

// the stream's handle, or torch's current one on the current device (raw: the queries of both, from torch._C)
void *stream_handle(PyObject *stream, PyObject *raw)
{
    PyObject *h;
    if (stream != Py_None) {
        h = PyObject_GetAttrString(stream, "cuda_stream");
    } else {
        if (!PyTuple_CheckExact(raw) || PyTuple_GET_SIZE(raw) != 2) throw Decline{};
        PyObject *dev = PyObject_CallNoArgs(PyTuple_GET_ITEM(raw, 1));
        if (!dev) { PyErr_Clear(); throw Decline{}; }
        h = PyObject_CallOneArg(PyTuple_GET_ITEM(raw, 0), dev);
        Py_DECREF(dev);
    }
    if (!h) { PyErr_Clear(); throw Decline{}; }
    void *p = nullptr;
    const bool ok = PyLong_CheckExact(h) && ((p = PyLong_AsVoidPtr(h)) || !PyErr_Occurred());
    Py_DECREF(h);
    if (!ok) { PyErr_Clear(); throw Decline{}; }
    return p;
}

template <typename F>
PyObject *guarded(Py_ssize_t given, Py_ssize_t wanted, F body)
{
    return ge_py::guarded(given, wanted, [&] {
        if (at::impl::torch_function_mode_enabled()) throw Decline{};
        return body();
    });
}

// (entry point, raw stream queries, M, N, K, A, lda, B, ldb, bias, alpha, act, C, ldc, batch, stream)
PyObject *plain(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded(n, 16, [&]() -> long {
        using Entry = ge_status_t (*)(int, int, int, const void *, int, const void *, int, const float *, float, ge_act_t, float *, int, int, void *);
        const Entry entry = (Entry)to_address(a[0]);
        const int M = to_int(a[2]), N = to_int(a[3]), K = to_int(a[4]), lda = to_int(a[6]), ldb = to_int(a[8]), ldc = to_int(a[13]), batch = to_int(a[14]);
        const at::Tensor *A = to_tensor(a[5]), *B = to_tensor(a[7]), *bias = to_tensor(a[9], true), *C = to_tensor(a[12]);
        const float alpha = to_float(a[10]);
        const int act = to_act(a[11]);
        extent(A, M, K, lda, batch);
        extent(B, K, N, ldb, batch);
        extent(C, M, N, ldc, batch);
        extent(bias, 1, N, N, 1);
        void *pa = address(A), *pb = address(B), *pbias = address(bias), *pc = address(C), *st = stream_handle(a[15], a[1]);
        return without_gil([&] { return entry(M, N, K, pa, lda, pb, ldb, (const float *)pbias, alpha, (ge_act_t)act, (float *)pc, ldc, batch, st); });
    });
}

// (entry point, raw stream queries, M, N, K, A, lda, B, ldb, C, ldc, batch, transA, transB, alpha, row_scale, bias, residual, ldr, beta, act, clamp, plan, split_k,
// workspace, stream, a_structure)
PyObject *fused(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded(n, 27, [&]() -> long {
        using Entry = ge_status_t (*)(const ge_fused_args_t *, void *);
        const Entry entry = (Entry)to_address(a[0]);
        ge_fused_args_t g{};
        g.M = to_int(a[2]); g.N = to_int(a[3]); g.K = to_int(a[4]);
        const at::Tensor *A = to_tensor(a[5]), *B = to_tensor(a[7]), *C = to_tensor(a[9]), *rowScale = to_tensor(a[15], true), *bias = to_tensor(a[16], true),
                         *R = to_tensor(a[17], true), *ws = to_tensor(a[24], true);
        g.lda = to_int(a[6]); g.ldb = to_int(a[8]); g.ldc = to_int(a[10]); g.batch = to_int(a[11]);
        g.transA = to_flag(a[12]); g.transB = to_flag(a[13]);
        g.alpha = to_float(a[14]);
        g.ldr = to_int(a[18]); g.beta = to_float(a[19]);
        g.act = (ge_act_t)to_act(a[20]);
        g.clamp_lo = -INFINITY; g.clamp_hi = INFINITY;
        if (a[21] != Py_None) {
            if (!PyTuple_CheckExact(a[21]) || PyTuple_GET_SIZE(a[21]) != 2) throw Decline{};
            g.clamp_lo = to_float(PyTuple_GET_ITEM(a[21], 0));
            g.clamp_hi = to_float(PyTuple_GET_ITEM(a[21], 1));
        }
        g.plan = (ge_plan_t)to_plan(a[22]);
        g.split_k = to_int(a[23]);
        g.a_structure = (decltype(g.a_structure))to_structure(a[26]);
        extent(A, g.transA ? g.K : g.M, g.transA ? g.M : g.K, g.lda, g.batch);
        extent(B, g.transB ? g.N : g.K, g.transB ? g.K : g.N, g.ldb, g.batch);
        extent(C, g.M, g.N, g.ldc, g.batch);
        extent(R, g.M, g.N, g.ldr, g.batch);
        extent(bias, 1, g.N, g.N, 1);
        extent(rowScale, 1, g.M, g.M, 1);
        g.A = (decltype(g.A))address(A); g.B = (decltype(g.B))address(B); g.C = address(C);
        g.row_scale = (const float *)address(rowScale); g.bias = (const float *)address(bias);
        g.R = address(R);
        g.r_type = (decltype(g.r_type))(R ? kind(R) : GE_DTYPE_F32);
        g.c_type = (decltype(g.c_type))kind(C);
        g.workspace = address(ws);
        g.workspace_bytes = ws ? (size_t)ws->numel() * ws->element_size() : 0;
        void *st = stream_handle(a[25], a[1]);
        return without_gil([&] { return entry(&g, st); });
    });
}

void pair(PyObject *o, int &first, int &second)
{
    if (!PyTuple_CheckExact(o) || PyTuple_GET_SIZE(o) < 2) throw Decline{};
    first = to_int(PyTuple_GET_ITEM(o, 0));
    second = to_int(PyTuple_GET_ITEM(o, 1));
}

// (entry point, raw stream queries, X, Wt, Y, stride, pad, dil, alpha, bias, residual, beta, act, clamp, workspace, stream)
PyObject *conv(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded(n, 16, [&]() -> long {
        using Entry = ge_status_t (*)(const ge_conv_args_t *, void *);
        const Entry entry = (Entry)to_address(a[0]);
        ge_conv_args_t g{};
        const at::Tensor *X = to_tensor(a[2]), *W = to_tensor(a[3]), *Y = to_tensor(a[4]), *bias = to_tensor(a[9], true), *R = to_tensor(a[10], true),
                         *ws = to_tensor(a[14], true);
        if (X->dim() != 4 || W->dim() != 4) throw Decline{};
        int *const xs[4] = {&g.N, &g.H, &g.W, &g.Cin};
        int inner = 0;                   // (the filters' channels are the input's, and not looked at)
        int *const ws4[4] = {&g.Cout, &g.KH, &g.KW, &inner};
        for (int i = 0; i < 4; ++i) {
            if (X->size(i) > INT_MAX || W->size(i) > INT_MAX) throw Decline{};
            *xs[i] = (int)X->size(i);
            *ws4[i] = (int)W->size(i);
        }
        pair(a[5], g.stride_h, g.stride_w);
        pair(a[6], g.pad_h, g.pad_w);
        pair(a[7], g.dil_h, g.dil_w);
        g.alpha = to_float(a[8]); g.beta = to_float(a[11]);
        g.act = (ge_act_t)to_act(a[12]);
        g.clamp_lo = -INFINITY; g.clamp_hi = INFINITY;
        if (a[13] != Py_None) {
            if (!PyTuple_CheckExact(a[13]) || PyTuple_GET_SIZE(a[13]) != 2) throw Decline{};
            g.clamp_lo = to_float(PyTuple_GET_ITEM(a[13], 0));
            g.clamp_hi = to_float(PyTuple_GET_ITEM(a[13], 1));
        }
        g.X = (decltype(g.X))address(X); g.Wt = (decltype(g.Wt))address(W); g.Y = address(Y);
        g.bias = (const float *)address(bias);
        g.R = address(R);
        g.r_type = (decltype(g.r_type))(R ? kind(R) : GE_DTYPE_F32);
        g.y_type = (decltype(g.y_type))kind(Y);
        g.workspace = address(ws);
        g.workspace_bytes = ws ? (size_t)ws->numel() * ws->element_size() : 0;
        void *st = stream_handle(a[15], a[1]);
        return without_gil([&] { return entry(&g, st); });
    });
}

// (entry point, raw stream queries, N, K, B, ldb, transB, bias, params, workspace, stream)
PyObject *rowsum_params(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded(n, 11, [&]() -> long {
        using Entry = ge_status_t (*)(int, int, const void *, int, int, const float *, float *, void *, size_t, void *);
        const Entry entry = (Entry)to_address(a[0]);
        const int N = to_int(a[2]), K = to_int(a[3]), ldb = to_int(a[5]), transB = to_flag(a[6]);
        const at::Tensor *B = to_tensor(a[4]), *bias = to_tensor(a[7], true), *params = to_tensor(a[8]), *ws = to_tensor(a[9], true);
        extent(B, transB ? N : K, transB ? K : N, ldb, 1);
        extent(params, 1, K + 1ll, K + 1ll, 1);
        void *pb = address(B), *pbias = address(bias), *pp = address(params), *pw = address(ws), *st = stream_handle(a[10], a[1]);
        const size_t bytes = ws ? (size_t)ws->numel() * ws->element_size() : 0;
        return without_gil([&] { return entry(N, K, pb, ldb, transB, (const float *)pbias, (float *)pp, pw, bytes, st); });
    });
}

// (entry point, raw stream queries, M, K, A, lda, params, alpha, y, stream)
PyObject *rowsum(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded(n, 10, [&]() -> long {
        using Entry = ge_status_t (*)(int, int, const void *, int, const float *, float, float *, void *);
        const Entry entry = (Entry)to_address(a[0]);
        const int M = to_int(a[2]), K = to_int(a[3]), lda = to_int(a[5]);
        const at::Tensor *A = to_tensor(a[4]), *params = to_tensor(a[6]), *y = to_tensor(a[8]);
        const float alpha = to_float(a[7]);
        void *pa = address(A), *pp = address(params), *py = address(y), *st = stream_handle(a[9], a[1]);
        return without_gil([&] { return entry(M, K, pa, lda, (const float *)pp, alpha, (float *)py, st); });
    });
}

PyMethodDef methods[] = {
    {"plain", (PyCFunction)(void (*)(void))plain, METH_FASTCALL, nullptr},
    {"fused", (PyCFunction)(void (*)(void))fused, METH_FASTCALL, nullptr},
    {"conv", (PyCFunction)(void (*)(void))conv, METH_FASTCALL, nullptr},
    {"rowsum_params", (PyCFunction)(void (*)(void))rowsum_params, METH_FASTCALL, nullptr},
    {"rowsum", (PyCFunction)(void (*)(void))rowsum, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// built_for: the torch whose headers this was compiled against (GE_TORCH_VERSION, from the build); binding.py takes it with no other
PyMODINIT_FUNC PyInit__marshal(void)
{
    PyObject *m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "built_for", GE_TORCH_VERSION) != 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
