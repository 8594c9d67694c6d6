// Native host path of the autograd wrapper: the same checks, allocations and
// library calls as paper_2608_10805_amd.binding and WTConvFunction, without
// the Python interpreter. A training step of a small layer was bound by them
// (14 x 14 B128 C384 L2 bf16: 98 us of kernels in a step of 242 us).
//
// apply() takes the plain case alone and returns None for every other one
// (anything the Python path converts, refuses or traces: see plain()); the
// caller then runs WTConvFunction, which converts, raises or traces as it does.
// The library's entry points come in as addresses (init), so this module
// links to torch only.
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/impl/LocalDispatchKeySet.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/custom_function.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/jit/frontend/tracer.h>
#include <torch/extension.h>

#include "wtconv.h"

namespace {

using at::Tensor;
using torch::autograd::AutogradContext;
using torch::autograd::variable_list;

decltype(&wtconv_forward_workspace_bytes) forward_bytes = nullptr;
decltype(&wtconv_forward) forward_fn = nullptr;
decltype(&wtconv_backward_workspace_bytes) backward_bytes = nullptr;
decltype(&wtconv_backward) backward_fn = nullptr;
PyObject* python_path = nullptr;  // autograd._backward
PyTypeObject* parameter_type = nullptr;  // torch.nn.Parameter

// A dense GPU tensor without wrappers (functorch, subclasses with a dispatch of
// their own) and without a forward-mode tangent.
bool plain(const Tensor& t, c10::Device dev)
{
    static const c10::DispatchKeySet wrapped(
        {c10::DispatchKey::Python, c10::DispatchKey::PythonTLSSnapshot, c10::DispatchKey::FuncTorchBatched,
         c10::DispatchKey::FuncTorchGradWrapper, c10::DispatchKey::Functionalize, c10::DispatchKey::Conjugate,
         c10::DispatchKey::Negative, c10::DispatchKey::ZeroTensor});
    return t.defined() && t.is_cuda() && t.device() == dev && t.layout() == at::kStrided && t.is_contiguous() &&
           !t.key_set().has_any(wrapped) && !t._fw_grad(0).defined();
}

bool param(const Tensor& t, c10::Device dev, at::IntArrayRef shape)
{
    return plain(t, dev) && t.scalar_type() == at::kFloat && t.sizes() == shape;
}

bool modes_active()
{
    const auto tls = c10::impl::tls_local_dispatch_key_set().included_;
    return torch::jit::tracer::isTracing() || c10::impl::TorchDispatchModeTLS::any_modes_set() ||
           tls.has(c10::DispatchKey::FuncTorchDynamicLayerFrontMode) || tls.has(c10::DispatchKey::Functionalize);
}

// The problem the arguments describe, if they are plain.
bool describe(const Tensor& x, const Tensor& bw, const Tensor& bs, const std::optional<Tensor>& bias,
              const variable_list& levels, wtconv_desc& d)
{
    if (!x.defined() || !x.is_cuda() || x.dim() != 4 || bw.dim() != 3 || levels.size() % 2) return false;
    const c10::Device dev = x.device();
    if (!plain(x, dev) || x.numel() == 0) return false;
    if (x.scalar_type() == at::kFloat)
        d.dtype = WTCONV_F32;
    else if (x.scalar_type() == at::kBFloat16)
        d.dtype = WTCONV_BF16;
    else if (x.scalar_type() == at::kHalf)
        d.dtype = WTCONV_F16;
    else
        return false;
    const int64_t C = x.size(1), k = bw.size(2), L = (int64_t)levels.size() / 2;
    for (int i = 0; i < 4; ++i)
        if (x.size(i) > INT_MAX) return false;
    if (k % 2 == 0 || k > WTCONV_MAX_KSIZE || L > WTCONV_MAX_LEVELS) return false;
    if (!param(bw, dev, {C, k, k}) || !param(bs, dev, {C})) return false;
    if (bias && !param(*bias, dev, {C})) return false;
    for (int64_t l = 0; l < L; ++l)
        if (!param(levels[l], dev, {4 * C, k, k}) || !param(levels[L + l], dev, {4 * C})) return false;
    d.B = (int)x.size(0);
    d.C = (int)C;
    d.H = (int)x.size(2);
    d.W = (int)x.size(3);
    d.k = (int)k;
    d.L = (int)L;
    return true;
}

void level_ptrs(const variable_list& levels, int L, const float** lw, const float** ls)
{
    for (int l = 0; l < L; ++l) {
        lw[l] = levels[l].const_data_ptr<float>();
        ls[l] = levels[L + l].const_data_ptr<float>();
    }
}

Tensor workspace(size_t bytes, const Tensor& like)
{
    return bytes ? at::empty({(int64_t)bytes}, like.options().dtype(at::kByte)) : Tensor();
}

struct Refused {
};  // the library refused the forward call

// The Python path's backward, for saved tensors or an upstream gradient that
// are not the plain case (saved-tensor hooks may hand back others) and for a
// call that the library refused: it converts them or raises as it does.
variable_list backward_in_python(const Tensor& x, const Tensor& dy, const Tensor& bw, const Tensor& bs,
                                 const std::optional<Tensor>& bias, const variable_list& levels, bool need_dx,
                                 bool need_db)
{
    py::gil_scoped_acquire gil;
    try {
        const py::object r =
            py::reinterpret_borrow<py::object>(python_path)(x, dy, bw, bs, bias, levels, need_dx, need_db);
        variable_list out;
        for (const py::handle& t : py::reinterpret_borrow<py::tuple>(r))
            out.push_back(t.is_none() ? Tensor() : t.cast<Tensor>());
        return out;
    } catch (py::error_already_set& e) {  // as the autograd engine hands Python errors on
        e.restore();
        python_error err;
        err.persist();
        throw python_error(std::move(err));
    }
}

struct Fn : public torch::autograd::Function<Fn> {
    // (the levels come one by one: autograd takes no list as a differentiable argument)
    template <typename... Levels>
    static Tensor forward(AutogradContext* ctx, const Tensor& x, const Tensor& bw, const Tensor& bs,
                          const std::optional<Tensor>& bias, const Levels&... level)
    {
        const variable_list levels = {level...};
        wtconv_desc d;
        TORCH_CHECK(describe(x, bw, bs, bias, levels, d), "wtconv: the arguments changed");
        Tensor y = at::empty_like(x);
        const size_t bytes = forward_bytes(&d);
        Tensor ws = workspace(bytes, x);
        const float *lw[WTCONV_MAX_LEVELS], *ls[WTCONV_MAX_LEVELS];
        level_ptrs(levels, d.L, lw, ls);
        const wtconv_status st =
            forward_fn(&d, x.const_data_ptr(), bw.const_data_ptr<float>(), bs.const_data_ptr<float>(),
                       bias ? bias->const_data_ptr<float>() : nullptr, d.L ? lw : nullptr, d.L ? ls : nullptr,
                       y.mutable_data_ptr(), bytes ? ws.mutable_data_ptr() : nullptr, bytes,
                       c10::hip::getCurrentHIPStream(x.device().index()));
        if (st != WTCONV_OK) throw Refused();
        variable_list saved = {x, bw, bs, bias ? *bias : Tensor()};
        saved.insert(saved.end(), levels.begin(), levels.end());
        ctx->save_for_backward(saved);
        return y;
    }

    static variable_list backward(AutogradContext* ctx, variable_list grads)
    {
        const variable_list saved = ctx->get_saved_variables();
        const Tensor &x = saved[0], &bw = saved[1], &bs = saved[2];
        std::optional<Tensor> bias;
        if (saved[3].defined()) bias = saved[3];
        const variable_list levels(saved.begin() + 4, saved.end());
        const bool need_dx = ctx->needs_input_grad(0), need_db = bias && ctx->needs_input_grad(3);
        wtconv_desc d;
        size_t bytes = 0;
        if (describe(x, bw, bs, bias, levels, d)) bytes = backward_bytes(&d);
        const Tensor dy = bytes ? grads[0].contiguous() : grads[0];
        if (!bytes || !dy.is_cuda() || dy.device() != x.device() || dy.scalar_type() != x.scalar_type() ||
            dy.sizes() != x.sizes())
            return backward_in_python(x, dy, bw, bs, bias, levels, need_dx, need_db);
        Tensor ws = workspace(bytes, x);
        variable_list out(4 + levels.size());
        if (need_dx) out[0] = at::empty_like(x);
        out[1] = at::empty_like(bw);
        out[2] = at::empty_like(bs);
        if (need_db) out[3] = at::empty_like(bs);
        for (size_t i = 0; i < levels.size(); ++i) out[4 + i] = at::empty_like(levels[i]);
        const float *lw[WTCONV_MAX_LEVELS], *ls[WTCONV_MAX_LEVELS];
        float *dlw[WTCONV_MAX_LEVELS], *dls[WTCONV_MAX_LEVELS];
        level_ptrs(levels, d.L, lw, ls);
        for (int l = 0; l < d.L; ++l) {
            dlw[l] = out[4 + l].mutable_data_ptr<float>();
            dls[l] = out[4 + d.L + l].mutable_data_ptr<float>();
        }
        const wtconv_status st = backward_fn(
            &d, x.const_data_ptr(), dy.const_data_ptr(), bw.const_data_ptr<float>(), bs.const_data_ptr<float>(),
            bias ? bias->const_data_ptr<float>() : nullptr, d.L ? lw : nullptr, d.L ? ls : nullptr,
            need_dx ? out[0].mutable_data_ptr() : nullptr, out[1].mutable_data_ptr<float>(),
            out[2].mutable_data_ptr<float>(), need_db ? out[3].mutable_data_ptr<float>() : nullptr,
            d.L ? dlw : nullptr, d.L ? dls : nullptr, ws.mutable_data_ptr(), bytes,
            c10::hip::getCurrentHIPStream(x.device().index()));
        if (st != WTCONV_OK) return backward_in_python(x, dy, bw, bs, bias, levels, need_dx, need_db);
        return out;
    }
};

template <size_t... I>
Tensor run(const Tensor& x, const Tensor& bw, const Tensor& bs, const std::optional<Tensor>& bias,
           const variable_list& levels, std::index_sequence<I...>)
{
    return Fn::apply(x, bw, bs, bias, levels[I]...);
}

template <size_t L = 0>
Tensor run(const Tensor& x, const Tensor& bw, const Tensor& bs, const std::optional<Tensor>& bias,
           const variable_list& levels)
{
    if (levels.size() == 2 * L) return run(x, bw, bs, bias, levels, std::make_index_sequence<2 * L>());
    if constexpr (L < WTCONV_MAX_LEVELS)
        return run<L + 1>(x, bw, bs, bias, levels);
    else
        throw Refused();
}

// A torch.Tensor or torch.nn.Parameter itself: other subclasses may override
// torch functions without a dispatch key that shows it.
bool exact_tensor(py::handle t)
{
    return Py_TYPE(t.ptr()) == reinterpret_cast<PyTypeObject*>(THPVariableClass) || Py_TYPE(t.ptr()) == parameter_type;
}

py::object apply(py::handle x, py::handle bw, py::handle bs, py::handle bias, py::sequence levels)
{
    if (!forward_fn || at::impl::torch_function_mode_enabled()) return py::none();
    if (!exact_tensor(x) || !exact_tensor(bw) || !exact_tensor(bs) || !(bias.is_none() || exact_tensor(bias)))
        return py::none();
    variable_list lv;
    lv.reserve(levels.size());
    for (const py::object& t : levels) {
        if (!exact_tensor(t)) return py::none();
        lv.push_back(THPVariable_Unpack(t.ptr()));
    }
    const Tensor &xt = THPVariable_Unpack(x.ptr()), &wt = THPVariable_Unpack(bw.ptr()), &st = THPVariable_Unpack(bs.ptr());
    std::optional<Tensor> bt;
    if (!bias.is_none()) bt = THPVariable_Unpack(bias.ptr());
    wtconv_desc d;
    if (modes_active() || !describe(xt, wt, st, bt, lv, d) || backward_bytes(&d) == 0) return py::none();
    Tensor y;
    try {
        py::gil_scoped_release no_gil;
        y = run(xt, wt, st, bt, lv);
    } catch (const Refused&) {
        return py::none();  // the Python path raises the library's error
    }
    return py::cast(y);
}

void init(uintptr_t fwd_bytes, uintptr_t fwd, uintptr_t bwd_bytes, uintptr_t bwd, py::object python_backward)
{
    forward_bytes = reinterpret_cast<decltype(forward_bytes)>(fwd_bytes);
    forward_fn = reinterpret_cast<decltype(forward_fn)>(fwd);
    backward_bytes = reinterpret_cast<decltype(backward_bytes)>(bwd_bytes);
    backward_fn = reinterpret_cast<decltype(backward_fn)>(bwd);
    py::object parameter = py::module_::import("torch.nn").attr("Parameter");
    parameter_type = reinterpret_cast<PyTypeObject*>(parameter.release().ptr());
    Py_XDECREF(python_path);
    python_path = python_backward.release().ptr();  // for the life of the process
}

}  // namespace

PYBIND11_MODULE(TORCH_EXTENSION_NAME, m)
{
    m.def("init", &init);
    m.def("apply", &apply);
}
