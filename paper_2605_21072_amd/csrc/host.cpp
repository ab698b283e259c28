// The online calls' marshalling in native code: argument checks, output and scratch tensors, the C entry point.  In Python (torch.empty
// twice, a ctypes call of twenty arguments) it took 4.7 us of the 12.9 that a linear costs the host, more than the GPU needs for
// the smallest shapes (two launches of 2.2 us each are the rest).  Calls with an explicit stream keep the Python path, which
// places memory in that stream's pool.  The functions return the entry point's status beside the tensors; the entry points' addresses come
// from the ctypes library, so that there is one copy of it.
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <torch/csrc/utils/pybind.h>

#include "../../include/qarvd.h"

namespace py = pybind11;
using OptTensor = std::optional<at::Tensor>;

namespace {

decltype(&qarvd_linear) linear_fn = nullptr;
decltype(&qarvd_linear_workspace) linear_workspace_fn = nullptr;
decltype(&qarvd_packed_ld) packed_ld_fn = nullptr;
decltype(&qarvd_quant_act) quant_act_fn = nullptr;
decltype(&qarvd_quant_act_static) quant_act_static_fn = nullptr;
decltype(&qarvd_w8a8_dual_gemm_variant) gemm_fn = nullptr;
decltype(&qarvd_w4a8_dual_gemm) gemm_w4_fn = nullptr;
decltype(&qarvd_w8a8_dual_gemm_q8) gemm_q8_fn = nullptr;

void init(const std::vector<uintptr_t> &a)
{
    linear_fn = reinterpret_cast<decltype(linear_fn)>(a.at(0));
    linear_workspace_fn = reinterpret_cast<decltype(linear_workspace_fn)>(a.at(1));
    packed_ld_fn = reinterpret_cast<decltype(packed_ld_fn)>(a.at(2));
    quant_act_fn = reinterpret_cast<decltype(quant_act_fn)>(a.at(3));
    quant_act_static_fn = reinterpret_cast<decltype(quant_act_static_fn)>(a.at(4));
    gemm_fn = reinterpret_cast<decltype(gemm_fn)>(a.at(5));
    gemm_w4_fn = reinterpret_cast<decltype(gemm_w4_fn)>(a.at(6));
    gemm_q8_fn = reinterpret_cast<decltype(gemm_q8_fn)>(a.at(7));
}

void *ptr(const OptTensor &t) { return t ? t->data_ptr() : nullptr; }

void check_2d(const at::Tensor &t, const char *what)
{
    if (!t.is_cuda() || t.dim() != 2 || t.stride(1) != 1)
        throw py::value_error(std::string(what) + " must be a 2-D device tensor with unit inner stride");
}

qarvd_dtype dtype_of(at::ScalarType s)
{
    if (s == at::kFloat) return QARVD_F32;
    if (s == at::kBFloat16) return QARVD_BF16;
    throw py::type_error("expected float32 or bfloat16, got " + std::string(py::str(py::cast(s))));
}

at::Tensor fresh(at::IntArrayRef size, at::ScalarType dtype, const at::Tensor &like)
{
    return at::empty(size, at::TensorOptions().dtype(dtype).device(like.device()));
}

// Runs a C entry point without the interpreter lock (a launch waits when the queue is full).
template <typename F> int run(F f)
{
    py::gil_scoped_release release;
    return (int)f();
}

py::tuple linear(const at::Tensor &X, const OptTensor &perm, int bits, const at::Tensor &Wq, const at::Tensor &sn, const at::Tensor &so,
                 const OptTensor &bias, int64_t N, int64_t K, int64_t K_o, std::optional<at::ScalarType> out_dtype, uintptr_t stream)
{
    check_2d(X, "X");
    const at::ScalarType out = c10::dtype_or_default(out_dtype);
    const int64_t M = X.size(0);
    if (X.size(1) != K)
        throw py::value_error("X has " + std::to_string(X.size(1)) + " channels, the layer " + std::to_string(K));
    const size_t need = linear_workspace_fn((int32_t)M, (int32_t)K, (int32_t)K_o);
    const at::Tensor ws = fresh({(int64_t)need}, at::kByte, X);
    at::Tensor Y = fresh({M, N}, out, X);
    const qarvd_dtype xdt = dtype_of(X.scalar_type()), ydt = dtype_of(out);
    const int st = run([&] {
        return linear_fn(X.data_ptr(), xdt, X.stride(0), (const int32_t *)ptr(perm), bits, Wq.data_ptr(), Wq.stride(0), (const float *)sn.data_ptr(),
                         (const float *)so.data_ptr(), (const float *)ptr(bias), (int32_t)M, (int32_t)N, (int32_t)K, (int32_t)K_o, Y.data_ptr(),
                         ydt, N, ws.data_ptr(), need, (void *)stream);
    });
    return py::make_tuple(st, std::move(Y));
}

py::tuple quant_act(const at::Tensor &X, const OptTensor &perm, int64_t K_o, OptTensor Xq, OptTensor s_x, uintptr_t stream)
{
    check_2d(X, "X");
    const int64_t M = X.size(0), K = X.size(1);
    if (!Xq) Xq = fresh({M, (int64_t)packed_ld_fn((int32_t)K, (int32_t)K_o)}, at::kChar, X);
    if (!s_x) s_x = fresh({M}, at::kFloat, X);
    const qarvd_dtype xdt = dtype_of(X.scalar_type());
    const int st = run([&] {
        return quant_act_fn(X.data_ptr(), xdt, (int32_t)M, (int32_t)K, X.stride(0), (const int32_t *)ptr(perm), (int32_t)K_o,
                            (int8_t *)Xq->data_ptr(), Xq->stride(0), (float *)s_x->data_ptr(), (void *)stream);
    });
    return py::make_tuple(st, std::move(Xq), std::move(s_x));
}

// The scale is required (None is a TypeError): a call without one must not become the per-token quantizer.
py::tuple quant_act_static(const at::Tensor &X, const OptTensor &perm, int64_t K_o, double scale, OptTensor Xq, uintptr_t stream)
{
    check_2d(X, "X");
    const int64_t M = X.size(0), K = X.size(1);
    if (!Xq) Xq = fresh({M, (int64_t)packed_ld_fn((int32_t)K, (int32_t)K_o)}, at::kChar, X);
    const qarvd_dtype xdt = dtype_of(X.scalar_type());
    const int st = run([&] {
        return quant_act_static_fn(X.data_ptr(), xdt, (int32_t)M, (int32_t)K, X.stride(0), (const int32_t *)ptr(perm), (int32_t)K_o, (float)scale,
                                   (int8_t *)Xq->data_ptr(), Xq->stride(0), (void *)stream);
    });
    return py::make_tuple(st, std::move(Xq));
}

// A vector that is missing (None) is refused by the entry point, with its status.
py::tuple gemm(const at::Tensor &Xq, const OptTensor &s_x, int bits, const at::Tensor &Wq, const OptTensor &sn, const OptTensor &so,
               const OptTensor &bias, int64_t M, int64_t N, int64_t K, int64_t K_o, std::optional<at::ScalarType> out_dtype, OptTensor Y,
               int variant, uintptr_t stream)
{
    if (!Y) Y = fresh({M, N}, c10::dtype_or_default(out_dtype), Xq);
    const qarvd_dtype ydt = dtype_of(Y->scalar_type());
    const int st = run([&] {
        if (bits == 4)
            return gemm_w4_fn((const int8_t *)Xq.data_ptr(), Xq.stride(0), (const float *)ptr(s_x), (const uint8_t *)Wq.data_ptr(), Wq.stride(0),
                              (const float *)ptr(sn), (const float *)ptr(so), (const float *)ptr(bias), (int32_t)M, (int32_t)N, (int32_t)K,
                              (int32_t)K_o, Y->data_ptr(), ydt, Y->stride(0), nullptr, nullptr, variant, (void *)stream);
        return gemm_fn(variant, (const int8_t *)Xq.data_ptr(), Xq.stride(0), (const float *)ptr(s_x), (const int8_t *)Wq.data_ptr(), Wq.stride(0),
                       (const float *)ptr(sn), (const float *)ptr(so), (const float *)ptr(bias), (int32_t)M, (int32_t)N, (int32_t)K,
                       (int32_t)K_o, Y->data_ptr(), ydt, Y->stride(0), nullptr, nullptr, (void *)stream);
    });
    return py::make_tuple(st, std::move(Y));
}

py::tuple gemm_q8(const at::Tensor &Xq, const OptTensor &s_x, const at::Tensor &Wq, const OptTensor &sn, const OptTensor &so, const OptTensor &bias,
                  int64_t M, int64_t N, int64_t K, int64_t K_o, double scale, int act, OptTensor Y8, int variant, uintptr_t stream)
{
    if (!Y8) Y8 = fresh({M, N}, at::kChar, Xq);
    const int st = run([&] {
        return gemm_q8_fn((const int8_t *)Xq.data_ptr(), Xq.stride(0), (const float *)ptr(s_x), (const int8_t *)Wq.data_ptr(), Wq.stride(0),
                          (const float *)ptr(sn), (const float *)ptr(so), (const float *)ptr(bias), (int32_t)M, (int32_t)N, (int32_t)K,
                          (int32_t)K_o, (qarvd_act)act, (float)scale, (int8_t *)Y8->data_ptr(), Y8->stride(0), variant, (void *)stream);
    });
    return py::make_tuple(st, std::move(Y8));
}

}  // namespace

PYBIND11_MODULE(_host, m)
{
    m.attr("torch_version") = QARVD_TORCH_VERSION;      // whose headers this was compiled against
    m.def("init", &init);
    m.def("linear", &linear);
    m.def("quant_act", &quant_act);
    m.def("quant_act_static", &quant_act_static);
    m.def("gemm", &gemm);
    m.def("gemm_q8", &gemm_q8);
}
