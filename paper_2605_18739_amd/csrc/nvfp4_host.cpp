// The binding's host path in native code: takes the pointers out of torch tensors, allocates what the caller did not
// hand over (output buffers, workspaces) and calls the C ABI of include/nvfp4.h.  Argument marshalling only, with the
// names of the C functions; binding.py holds the Python signatures.
//
// A small call is bound by this work, not by its kernels: through ctypes and torch.empty a quantizer call spent 15.5 us
// on the host (three output buffers and a workspace 6.6, the current stream 2.9, argument objects 2.5, the launch 3.4),
// of which the launch and four allocations at 0.5 us each remain.
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <torch/csrc/Device.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/version.h>

#include <algorithm>
#include <vector>

#include "../../include/nvfp4.h"

namespace {

PyObject *s_codes, *s_scales, *s_global_scale, *s_rows, *s_K;      // attribute names

struct Fail {};                                                     // a Python error has been set

void fail(PyObject *type, const char *text)
{
    PyErr_SetString(type, text);
    throw Fail();
}
void require(bool ok, const char *text)
{
    if (!ok) fail(PyExc_AssertionError, text);
}

const at::Tensor &tensor(PyObject *o)
{
    if (!THPVariable_Check(o)) fail(PyExc_TypeError, "expected a torch.Tensor");
    return THPVariable_Unpack(o);
}
void *address(PyObject *o) { return o == Py_None ? nullptr : tensor(o).data_ptr(); }

long long number(PyObject *o)
{
    const long long v = PyLong_AsLongLong(o);
    if (v == -1 && PyErr_Occurred()) throw Fail();
    return v;
}
void *stream_of(PyObject *o)
{
    void *p = PyLong_AsVoidPtr(o);
    if (!p && PyErr_Occurred()) throw Fail();
    return p;
}

PyObject *attribute(PyObject *o, PyObject *name)                    // (borrowed by the caller for as long as o keeps it)
{
    PyObject *a = PyObject_GetAttr(o, name);
    if (!a) throw Fail();
    return a;
}

// An NVFP4Tensor; holds references, so the buffers live through the call whatever other threads do to the object (what
// stands in the argument list itself is held by the caller)
struct Quantized {
    nvfp4_tensor t{};
    at::Tensor codes, scales, global_scale;
    explicit Quantized(PyObject *o)
    {
        t.codes = static_cast<uint8_t *>(buffer(o, s_codes, codes));
        t.scales = static_cast<uint8_t *>(buffer(o, s_scales, scales));
        t.global_scale = static_cast<float *>(buffer(o, s_global_scale, global_scale));
        t.rows = count(o, s_rows);
        t.K = count(o, s_K);
    }
    nvfp4_tensor *c() { return &t; }

private:
    static void *buffer(PyObject *o, PyObject *name, at::Tensor &keep)
    {
        PyObject *a = attribute(o, name);
        const bool is = THPVariable_Check(a);
        if (is) keep = THPVariable_Unpack(a);
        Py_DECREF(a);
        if (!is) fail(PyExc_TypeError, "expected an NVFP4Tensor");
        return keep.data_ptr();
    }
    static int64_t count(PyObject *o, PyObject *name)
    {
        PyObject *a = attribute(o, name);
        const long long v = PyLong_AsLongLong(a);
        Py_DECREF(a);
        if (v == -1 && PyErr_Occurred()) throw Fail();
        return v;
    }
};

at::Tensor bytes_on(const at::Device &device, int64_t n) { return at::empty({n}, at::TensorOptions().device(device).dtype(at::kByte)); }

// the caller's workspace, or one for this call: from the current stream's pool, and back to it when the call returns,
// behind the launches.  So the stream of a call without a workspace is torch's current one (binding.py sees to it).
struct Workspace {
    at::Tensor t;
    Workspace(PyObject *given, const at::Device &device, int op, int64_t a, int64_t b, int64_t c = 0)
    {
        if (given != Py_None) t = tensor(given);
        else t = bytes_on(device, std::max<int64_t>(16, (int64_t)nvfp4_workspace_bytes(op, a, b, c)));
    }
    void *data() const { return t.data_ptr(); }
    size_t size() const { return (size_t)t.numel(); }
};

// the library may wait for a lock: not under the GIL, which is taken again however the call ends (what torch throws
// while the arguments of the call are put together becomes a Python error)
struct WithoutGil {
    PyThreadState *saved = PyEval_SaveThread();
    ~WithoutGil() { PyEval_RestoreThread(saved); }
};
template <class F>
PyObject *status(F &&call)
{
    int rc;
    {
        WithoutGil released;
        rc = call();
    }
    return PyLong_FromLong(rc);
}

const at::Tensor &matrix(PyObject *o)
{
    const at::Tensor &x = tensor(o);
    require(x.scalar_type() == at::kBFloat16 && x.dim() == 2 && x.stride(1) == 1, "expected a bf16 matrix with unit stride along its rows");
    return x;
}
const at::Tensor &heads(PyObject *o)
{
    const at::Tensor &x = tensor(o);
    require(x.scalar_type() == at::kBFloat16 && x.dim() == 3 && x.is_contiguous(), "expected a contiguous bf16 tensor [T, H, d]");
    return x;
}

// ---- allocation -------------------------------------------------------------------------------------
// buffers(rows, K, device) -> codes [rows, K/2] u8, scales [rows, K/16] u8, global_scale [1] f32
PyObject *buffers(PyObject *const *a)
{
    const int64_t rows = number(a[0]), K = number(a[1]);
    const at::Device device = ((THPDevice *)a[2])->device;
    const auto bytes = at::TensorOptions().device(device).dtype(at::kByte);
    PyObject *r = PyTuple_New(3);
    if (!r) throw Fail();
    try {
        PyTuple_SET_ITEM(r, 0, THPVariable_Wrap(at::empty({rows, K / 2}, bytes)));
        PyTuple_SET_ITEM(r, 1, THPVariable_Wrap(at::empty({rows, K / 16}, bytes)));
        PyTuple_SET_ITEM(r, 2, THPVariable_Wrap(at::empty({1}, bytes.dtype(at::kFloat))));
    } catch (...) {
        Py_DECREF(r);
        throw;
    }
    return r;
}
// output(like, M, N, is_bf16) -> [M, N] beside `like`
PyObject *output(PyObject *const *a)
{
    return THPVariable_Wrap(at::empty({number(a[1]), number(a[2])},
                                      at::TensorOptions().device(tensor(a[0]).device()).dtype(a[3] == Py_True ? at::kBFloat16 : at::kFloat)));
}

// ---- quantizers: (x, ..., out, workspace, stream) -----------------------------------------------------
PyObject *quantize(PyObject *const *a)                              // x, block_axis, scale, out, workspace, stream
{
    const at::Tensor &x = matrix(a[0]);
    const int axis = (int)number(a[1]);
    Quantized out(a[3]);
    Workspace ws(a[4], x.device(), NVFP4_OP_QUANTIZE, x.size(0), x.size(1));
    const float *scale = static_cast<const float *>(address(a[2]));
    void *s = stream_of(a[5]), *p = x.data_ptr();
    return status([&] { return nvfp4_quantize(p, x.size(0), x.size(1), x.stride(0), axis, scale, out.c(), ws.data(), ws.size(), s); });
}
PyObject *quantize_4over6(PyObject *const *a)                       // x, scale, out, workspace, stream
{
    const at::Tensor &x = matrix(a[0]);
    Quantized out(a[2]);
    Workspace ws(a[3], x.device(), NVFP4_OP_QUANTIZE_4OVER6, x.size(0), x.size(1));
    const float *scale = static_cast<const float *>(address(a[1]));
    void *s = stream_of(a[4]), *p = x.data_ptr();
    return status([&] { return nvfp4_quantize_4over6(p, x.size(0), x.size(1), x.stride(0), scale, out.c(), ws.data(), ws.size(), s); });
}
PyObject *quantize_rht(PyObject *const *a)                          // x, sign_mask, scale, out, workspace, stream
{
    const at::Tensor &x = matrix(a[0]);
    const uint32_t mask = (uint32_t)number(a[1]);
    Quantized out(a[3]);
    Workspace ws(a[4], x.device(), NVFP4_OP_QUANTIZE_RHT, x.size(0), x.size(1));
    const float *scale = static_cast<const float *>(address(a[2]));
    void *s = stream_of(a[5]), *p = x.data_ptr();
    return status([&] { return nvfp4_quantize_rht(p, x.size(0), x.size(1), x.stride(0), mask, scale, out.c(), ws.data(), ws.size(), s); });
}
PyObject *quantize_2d(PyObject *const *a)                           // w, scale, out, out_t or None, workspace, stream
{
    const at::Tensor &w = matrix(a[0]);
    Quantized out(a[2]);
    const bool transposed = a[3] != Py_None;
    Quantized out_t(transposed ? a[3] : a[2]);
    Workspace ws(a[4], w.device(), NVFP4_OP_QUANTIZE_2D, w.size(0), w.size(1));
    const float *scale = static_cast<const float *>(address(a[1]));
    void *s = stream_of(a[5]), *p = w.data_ptr();
    return status([&] { return nvfp4_quantize_2d(p, w.size(0), w.size(1), w.stride(0), scale, out.c(), transposed ? out_t.c() : nullptr, ws.data(), ws.size(), s); });
}
PyObject *quantize_for_all_to_all(PyObject *const *a)               // x, P, scale, out, workspace, stream
{
    const at::Tensor &x = heads(a[0]);
    const int64_t P = number(a[1]);
    Quantized out(a[3]);
    Workspace ws(a[4], x.device(), NVFP4_OP_QUANTIZE_A2A, x.size(0), x.size(1), x.size(2));
    const float *scale = static_cast<const float *>(address(a[2]));
    void *s = stream_of(a[5]), *p = x.data_ptr();
    return status([&] { return nvfp4_quantize_for_all_to_all(p, x.size(0), x.size(1), x.size(2), P, scale, out.c(), ws.data(), ws.size(), s); });
}

// ---- KV cache -----------------------------------------------------------------------------------------
template <int OP, class F>
PyObject *kv_write(PyObject *const *a, F f)                         // kv, out, workspace, stream
{
    const at::Tensor &x = heads(a[0]);
    Quantized out(a[1]);
    Workspace ws(a[2], x.device(), OP, x.size(0), x.size(1), x.size(2));
    void *s = stream_of(a[3]), *p = x.data_ptr();
    return status([&] { return f(p, x.size(0), x.size(1), x.size(2), out.c(), ws.data(), ws.size(), s); });
}
PyObject *kv_quant(PyObject *const *a) { return kv_write<NVFP4_OP_KV_QUANT>(a, nvfp4_kv_quant); }
PyObject *kv_quant_4over6(PyObject *const *a) { return kv_write<NVFP4_OP_KV_QUANT_4OVER6>(a, nvfp4_kv_quant_4over6); }
PyObject *kv_quant_noalloc(PyObject *const *a)                      // kv, out, stream
{
    const at::Tensor &x = heads(a[0]);
    Quantized out(a[1]);
    void *s = stream_of(a[2]), *p = x.data_ptr();
    return status([&] { return nvfp4_kv_quant_noalloc(p, x.size(0), x.size(1), x.size(2), out.c(), s); });
}
PyObject *kv_quant_k(PyObject *const *a)                            // k, out, row_mean, workspace, stream
{
    const at::Tensor &x = heads(a[0]);
    Quantized out(a[1]);
    Workspace ws(a[3], x.device(), NVFP4_OP_KV_QUANT_K, x.size(0), x.size(1), x.size(2));
    void *mean = address(a[2]), *s = stream_of(a[4]), *p = x.data_ptr();
    return status([&] { return nvfp4_kv_quant_k(p, x.size(0), x.size(1), x.size(2), out.c(), mean, ws.data(), ws.size(), s); });
}
PyObject *kv_dequant(PyObject *const *a)                            // q, T, H, d, out, stream
{
    Quantized q(a[0]);
    const int64_t T = number(a[1]), H = number(a[2]), d = number(a[3]);
    void *out = address(a[4]), *s = stream_of(a[5]);
    return status([&] { return nvfp4_kv_dequant(q.c(), out, T, H, d, s); });
}
PyObject *kv_dequant_gather(PyObject *const *a)                     // [(q, row_mean or None, T), ...], H, d, out, stream
{
    // tuples of our own: a list may change under the call (attributes are read on the way, and the GIL is released)
    struct Owned {
        PyObject *o;
        explicit Owned(PyObject *sequence) : o(PySequence_Tuple(sequence))
        {
            if (!o) throw Fail();
        }
        Owned(const Owned &) = delete;
        ~Owned() { Py_DECREF(o); }
    } seq(a[0]);
    const Py_ssize_t n = PyTuple_GET_SIZE(seq.o);
    std::vector<nvfp4_kv_chunk> chunks((size_t)std::max<Py_ssize_t>(n, 1));     // (an empty list is refused for its size, not as a null pointer)
    std::vector<Quantized> keep;
    std::vector<at::Tensor> keep_means;
    keep.reserve((size_t)n);
    keep_means.reserve((size_t)n);
    for (Py_ssize_t i = 0; i < n; ++i) {
        const Owned c(PyTuple_GET_ITEM(seq.o, i));
        if (PyTuple_GET_SIZE(c.o) != 3) fail(PyExc_ValueError, "a chunk is (NVFP4Tensor, row_mean or None, T)");
        PyObject *mean = PyTuple_GET_ITEM(c.o, 1);
        keep.emplace_back(PyTuple_GET_ITEM(c.o, 0));
        if (mean != Py_None) keep_means.push_back(tensor(mean));
        chunks[(size_t)i] = {keep.back().t, address(mean), number(PyTuple_GET_ITEM(c.o, 2))};
    }
    const int64_t H = number(a[1]), d = number(a[2]);
    void *out = address(a[3]), *s = stream_of(a[4]);
    return status([&] { return nvfp4_kv_dequant_gather(chunks.data(), (int)n, out, H, d, s); });
}

// ---- GEMMs --------------------------------------------------------------------------------------------
PyObject *gemm(PyObject *const *a)                                  // A, W, out_dtype, Y, stream
{
    Quantized A(a[0]), W(a[1]);
    const int dtype = (int)number(a[2]);
    const at::Tensor &Y = tensor(a[3]);
    void *s = stream_of(a[4]), *p = Y.data_ptr();
    return status([&] { return nvfp4_gemm(A.c(), W.c(), p, Y.stride(0), dtype, s); });
}
PyObject *gemm_scale_out(PyObject *const *a)                        // A, W, Y, scale_out, workspace, stream
{
    Quantized A(a[0]), W(a[1]);
    const at::Tensor &Y = tensor(a[2]);
    Workspace ws(a[4], A.codes.device(), NVFP4_OP_GEMM_SCALE_OUT, A.t.rows, W.t.rows);
    float *scale = static_cast<float *>(address(a[3]));
    void *s = stream_of(a[5]), *p = Y.data_ptr();
    return status([&] { return nvfp4_gemm_scale_out(A.c(), W.c(), p, Y.stride(0), scale, ws.data(), ws.size(), s); });
}
PyObject *lora_down(PyObject *const *a)                             // x, a, t, workspace, stream
{
    const at::Tensor &x = matrix(a[0]), &f = tensor(a[1]);
    require(f.scalar_type() == at::kBFloat16 && f.is_contiguous() && f.dim() == 2 && f.size(0) == NVFP4_LORA_RANK && f.size(1) == x.size(1),
            "expected a contiguous bf16 factor [128, K]");
    Workspace ws(a[3], x.device(), NVFP4_OP_LORA_DOWN, x.size(0), x.size(1));
    void *t = address(a[2]), *s = stream_of(a[4]), *p = x.data_ptr(), *pa = f.data_ptr();
    return status([&] { return nvfp4_lora_down(p, x.size(0), x.size(1), x.stride(0), pa, t, ws.data(), ws.size(), s); });
}
PyObject *gemm_lora(PyObject *const *a)                             // A, W, t, b, lora_scale, out_dtype, Y, stream
{
    Quantized A(a[0]), W(a[1]);
    const at::Tensor &t = tensor(a[2]), &b = tensor(a[3]), &Y = tensor(a[6]);
    require(t.is_contiguous() && b.is_contiguous() && t.dim() == 2 && b.dim() == 2 && t.size(0) == A.t.rows && b.size(0) == W.t.rows &&
                t.size(1) == NVFP4_LORA_RANK && b.size(1) == NVFP4_LORA_RANK,
            "expected contiguous factors t [M, 128] and b [N, 128]");
    const double scale = PyFloat_AsDouble(a[4]);
    if (scale == -1.0 && PyErr_Occurred()) throw Fail();
    const int dtype = (int)number(a[5]);
    void *s = stream_of(a[7]), *pt = t.data_ptr(), *pb = b.data_ptr(), *py = Y.data_ptr();
    return status([&] { return nvfp4_gemm_lora(A.c(), W.c(), pt, pb, (float)scale, py, Y.stride(0), dtype, s); });
}
PyObject *gemm_act_quant(PyObject *const *a)                        // A, W, act, scale, out, h_bf16, workspace, stream
{
    Quantized A(a[0]), W(a[1]), out(a[4]);
    const int act = (int)number(a[2]);
    const float *scale = static_cast<const float *>(address(a[3]));
    void *h = address(a[5]);
    const int flags = (h ? 1 : 0) | ((scale && A.t.K % 64 == 0) ? 2 : 0);
    Workspace ws(a[6], A.codes.device(), NVFP4_OP_GEMM_ACT_QUANT, A.t.rows, W.t.rows, flags);
    void *s = stream_of(a[7]);
    return status([&] { return nvfp4_gemm_act_quant(A.c(), W.c(), act, scale, out.c(), h, ws.data(), ws.size(), s); });
}

// one Python function: fixed number of positional arguments, C++ and torch exceptions turned into Python's
template <PyObject *(*F)(PyObject *const *), int N>
PyObject *entry(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != N) {
        PyErr_Format(PyExc_TypeError, "%d arguments expected, %zd given", N, n);
        return nullptr;
    }
    try {
        return F(args);
    } catch (const Fail &) {
        return nullptr;
    }
    END_HANDLE_TH_ERRORS
}
template <PyObject *(*F)(PyObject *const *), int N>
constexpr PyMethodDef method(const char *name)
{
    return {name, (PyCFunction)(void (*)(void))entry<F, N>, METH_FASTCALL, nullptr};
}

}  // namespace

extern "C" PyObject *PyInit__host(void)
{
    static PyMethodDef methods[] = {
        method<buffers, 3>("buffers"), method<output, 4>("output"), method<quantize, 6>("quantize"),
        method<quantize_4over6, 5>("quantize_4over6"), method<quantize_rht, 6>("quantize_rht"), method<quantize_2d, 6>("quantize_2d"),
        method<quantize_for_all_to_all, 6>("quantize_for_all_to_all"), method<kv_quant, 4>("kv_quant"),
        method<kv_quant_4over6, 4>("kv_quant_4over6"), method<kv_quant_noalloc, 3>("kv_quant_noalloc"), method<kv_quant_k, 5>("kv_quant_k"),
        method<kv_dequant, 6>("kv_dequant"), method<kv_dequant_gather, 5>("kv_dequant_gather"), method<gemm, 5>("gemm"),
        method<gemm_scale_out, 6>("gemm_scale_out"), method<lora_down, 5>("lora_down"), method<gemm_lora, 8>("gemm_lora"),
        method<gemm_act_quant, 8>("gemm_act_quant"), {nullptr, nullptr, 0, nullptr}};
    static PyModuleDef module = {PyModuleDef_HEAD_INIT, "_host", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};
    s_codes = PyUnicode_InternFromString("codes");
    s_scales = PyUnicode_InternFromString("scales");
    s_global_scale = PyUnicode_InternFromString("global_scale");
    s_rows = PyUnicode_InternFromString("rows");
    s_K = PyUnicode_InternFromString("K");
    PyObject *m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "torch_version", TORCH_VERSION) != 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
