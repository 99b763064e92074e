// Autograd nodes of the KAN and UKAN layers over the C ABI of libkan_hip.so (include/kan.h).
//
// Nothing is computed here: forward calls kan_forward_kept / ukan_cg_forward_saved, backward calls kan_backward_saved /
// ukan_cg_backward_saved with exactly the gradients autograd asks for.  Native, because a step of a small network is bound by
// the host: with the nodes in Python and the calls through ctypes a step of the [2, 5, 1] network took 230 .. 330 us for 80 us
// of GPU work, and a layer's backward node needs the interpreter lock here no more.  Tensors of a forward pass are kept
// through save_for_backward only, so hooks on saved tensors and the checks for changes in place see them.
#include <torch/csrc/autograd/custom_function.h>
#include <torch/csrc/jit/frontend/tracer.h>
#include <torch/csrc/utils/pybind.h>
#include <torch/library.h>
#include <ATen/ops/empty.h>
#include <c10/hip/HIPStream.h>
#include "kan.h"

namespace {

using at::Tensor;
using torch::autograd::AutogradContext;
using torch::autograd::variable_list;

[[noreturn]] void raise_kan_error(int status, const char *where)
{
    py::gil_scoped_acquire lock;
    const py::object type = py::module_::import("paper_2408_11200_amd.binding").attr("KanError");
    PyErr_SetObject(type.ptr(), type(status, where).ptr());
    throw py::error_already_set();
}

void check(int status, const char *where)
{
    if (status != KAN_OK) raise_kan_error(status, where);
}

[[noreturn]] void refuse(const char *what)
{
    py::gil_scoped_acquire lock;
    PyErr_SetString(PyExc_AssertionError, what);
    throw py::error_already_set();
}

// pointer of a device-resident contiguous fp32 tensor (null: no tensor); anything else is refused as binding.py refuses it
float *f32(const Tensor &t)
{
    if (!t.defined()) return nullptr;
    if (t.scalar_type() != at::kFloat || !t.is_cuda() || !t.is_contiguous()) refuse("device-resident contiguous float32 tensors only");
    return static_cast<float *>(t.data_ptr());
}

// What a forward pass left for its backward pass, as the graph hands it back: a hook on saved tensors may have replaced it.
void *kept(const Tensor &t)
{
    if (!t.is_cuda() || !t.is_contiguous()) refuse("device-resident contiguous tensors only");
    return t.data_ptr();
}

Tensor or_none(const std::optional<Tensor> &t) { return t ? *t : Tensor(); }

Tensor whole(const Tensor &t) { return t.defined() ? t.contiguous() : t; }

// the current device's current stream: during backward the one of the forward pass, which the engine has set
void *stream() { return (void *)c10::hip::getCurrentHIPStream().stream(); }

Tensor bytes_like(const Tensor &x, size_t n) { return at::empty({(int64_t)(n > 256 ? n : 256)}, x.options().dtype(at::kByte)); }

// A struct of plain values carried from forward to backward.
template <class T>
c10::IValue pack(const T &v) { return std::string(reinterpret_cast<const char *>(&v), sizeof(T)); }
template <class T>
T unpack(const c10::IValue &v)
{
    T t;
    std::memcpy(&t, v.toStringRef().data(), sizeof(T));
    return t;
}

struct KanLayer : torch::autograd::Function<KanLayer> {
    static Tensor forward(AutogradContext *ctx, const Tensor &x, const Tensor &coef, const Tensor &w_s,
                          const std::optional<Tensor> &base, kan_layer_desc d)
    {
        const Tensor w_b = or_none(base);
        const int64_t B = x.size(0);
        // the scale-folded table is handed to the backward pass, the rest of the workspace is not
        const size_t kept = kan_workspace_bytes(&d, 0, KAN_PASS_FORWARD), whole_ws = kan_workspace_bytes(&d, B, KAN_PASS_FORWARD);
        const Tensor table = bytes_like(x, kept), ws = whole_ws > kept ? bytes_like(x, whole_ws - kept) : Tensor();
        ctx->saved_data["desc"] = pack(d);
        ctx->save_for_backward({x, coef, w_s, w_b, table});
        const Tensor y = at::empty({B, d.n_out}, x.options().dtype(at::kFloat));
        const Tensor xc = whole(x), cc = whole(coef), sc = whole(w_s), bc = whole(w_b);
        check(kan_forward_kept(&d, B, f32(xc), f32(cc), f32(sc), f32(bc), f32(y), table.data_ptr(), (size_t)table.numel(),
                               ws.defined() ? ws.data_ptr() : nullptr, ws.defined() ? (size_t)ws.numel() : 0, stream()),
              "kan_forward");
        return y;
    }

    static variable_list backward(AutogradContext *ctx, variable_list grads)
    {
        const kan_layer_desc d = unpack<kan_layer_desc>(ctx->saved_data["desc"]);
        const variable_list saved = ctx->get_saved_variables();
        const Tensor xc = whole(saved[0]), cc = whole(saved[1]), sc = whole(saved[2]), bc = whole(saved[3]), &table = saved[4];
        const int64_t B = xc.size(0);
        // edges: x, coef, w_s, and w_b if there is one
        const bool need[4] = {ctx->needs_input_grad(0), ctx->needs_input_grad(1), ctx->needs_input_grad(2),
                              bc.defined() && ctx->needs_input_grad(3)};
        variable_list g(5);
        if (!(need[0] || need[1] || need[2] || need[3])) return g;
        const Tensor gy = whole(grads[0]);
        const auto f = xc.options().dtype(at::kFloat);
        if (need[0]) g[0] = at::empty({B, d.n_in}, f);
        if (need[1]) g[1] = at::empty({d.n_in, d.G + d.k, d.n_out}, f);
        if (need[2]) g[2] = at::empty({d.n_in, d.n_out}, f);
        if (need[3]) g[3] = at::empty({d.n_in, d.n_out}, f);
        const Tensor bws = bytes_like(xc, kan_workspace_bytes(&d, B, KAN_PASS_BACKWARD));
        check(kan_backward_saved(&d, B, f32(xc), f32(cc), f32(sc), f32(bc), f32(gy), kept(table), f32(g[0]), f32(g[1]), f32(g[2]),
                                 f32(g[3]), bws.data_ptr(), (size_t)bws.numel(), stream()),
              "kan_backward_saved");
        return g;
    }
};

struct UkanCall {
    ukan_layer_desc d;
    int32_t max_groups, span;
};

ukan_params params_of(const Tensor (&p)[7])
{
    return ukan_params{f32(p[0]), f32(p[1]), f32(p[2]), f32(p[3]), f32(p[4]), f32(p[5]), f32(p[6])};
}

struct UkanLayer : torch::autograd::Function<UkanLayer> {
    static Tensor forward(AutogradContext *ctx, const Tensor &x, const Tensor &E, const Tensor &W1, const Tensor &b1, const Tensor &W2,
                          const Tensor &b2, const Tensor &scale, const std::optional<Tensor> &base, UkanCall c)
    {
        const Tensor w_b = or_none(base);
        const int64_t B = x.size(0);
        const Tensor y = at::empty({B, c.d.n_out}, x.options().dtype(at::kFloat));
        const Tensor saved = bytes_like(x, ukan_saved_bytes(&c.d, c.max_groups));
        const Tensor ws = bytes_like(x, ukan_workspace_bytes(&c.d, B, c.max_groups, KAN_PASS_FORWARD));
        const Tensor xc = whole(x);
        const Tensor tensors[7] = {E, W1, b1, W2, b2, scale, w_b};
        const ukan_params p = params_of(tensors);
        check(ukan_cg_forward_saved(&c.d, B, f32(xc), &p, f32(y), c.max_groups, saved.data_ptr(), (size_t)saved.numel(), &c.span,
                                    ws.data_ptr(), (size_t)ws.numel(), stream()),
              "ukan_cg_forward_saved");
        ctx->saved_data["call"] = pack(c);
        ctx->save_for_backward({x, E, W1, b1, W2, b2, scale, w_b, saved});
        return y;
    }

    static variable_list backward(AutogradContext *ctx, variable_list grads)
    {
        const UkanCall c = unpack<UkanCall>(ctx->saved_data["call"]);
        const variable_list saved = ctx->get_saved_variables();
        const Tensor xc = whole(saved[0]), &held = saved[8];
        const Tensor tensors[7] = {saved[1], saved[2], saved[3], saved[4], saved[5], saved[6], saved[7]};
        const int64_t B = xc.size(0), K = c.d.k + 1, dz = c.d.d_feat + c.d.d_pe;
        variable_list g(9);
        const auto f = xc.options().dtype(at::kFloat);
        const std::vector<int64_t> shapes[8] = {{B, c.d.n_in},          {c.d.n_in, c.d.d_feat}, {dz, c.d.d_hidden},    {c.d.d_hidden},
                                                {c.d.d_hidden, K * c.d.n_out}, {K * c.d.n_out}, {c.d.n_in, c.d.n_out}, {c.d.n_in, c.d.n_out}};
        bool any = false;
        for (int i = 0; i < 8; ++i) {
            if (i == 7 && !tensors[6].defined()) break;
            if (!ctx->needs_input_grad((size_t)i)) continue;
            g[i] = at::empty(shapes[i], f);
            any = true;
        }
        if (!any) return g;
        const Tensor gy = whole(grads[0]);
        const ukan_params p = params_of(tensors);
        const ukan_grads gg = {f32(g[1]), f32(g[2]), f32(g[3]), f32(g[4]), f32(g[5]), f32(g[6]), f32(g[7])};
        const Tensor ws = bytes_like(xc, ukan_workspace_bytes(&c.d, B, c.max_groups, KAN_PASS_BACKWARD));
        check(ukan_cg_backward_saved(&c.d, B, f32(xc), &p, f32(gy), f32(g[0]), &gg, c.max_groups, kept(held), (size_t)held.numel(),
                                     c.span, ws.data_ptr(), (size_t)ws.numel(), stream()),
              "ukan_cg_backward_saved");
        return g;
    }
};

Tensor kan_layer(const Tensor &x, const Tensor &coef, const Tensor &w_s, const std::optional<Tensor> &w_b, int64_t n_in, int64_t n_out,
                 int64_t G, int64_t k, double lo, double hi, int64_t base_act)
{
    const kan_layer_desc d = {(int32_t)n_in, (int32_t)n_out, (int32_t)G, (int32_t)k, (float)lo, (float)hi, (int32_t)base_act};
    return KanLayer::apply(x, coef, w_s, w_b, d);
}

Tensor ukan_layer(const Tensor &x, const Tensor &E, const Tensor &W1, const Tensor &b1, const Tensor &W2, const Tensor &b2,
                  const Tensor &scale, const std::optional<Tensor> &w_b, int64_t n_in, int64_t n_out, int64_t k, double h, int64_t d_pe,
                  int64_t d_feat, int64_t d_hidden, int64_t base_act, int64_t max_groups)
{
    const UkanCall c = {{(int32_t)n_in, (int32_t)n_out, (int32_t)k, (float)h, (int32_t)d_pe, (int32_t)d_feat, (int32_t)d_hidden,
                         (int32_t)base_act}, (int32_t)max_groups, 0};
    return UkanLayer::apply(x, E, W1, b1, W2, b2, scale, w_b, c);
}

// The layers as operators of torch's dispatcher: what torch.jit.trace records.  It sees dispatched calls only, so a node applied
// directly would leave nothing in the graph but the allocation of its result.  Outside a trace the dispatcher is passed by.
constexpr const char *kKanOp = "paper_2408_11200_amd::kan_layer", *kUkanOp = "paper_2408_11200_amd::ukan_layer";

template <class F, class... A>
Tensor call(const char *op, F f, const A &...a)
{
    py::gil_scoped_release unlock;
    if (!torch::jit::tracer::isTracing()) return f(a...);
    return c10::Dispatcher::singleton().findSchemaOrThrow(op, "").typed<std::remove_pointer_t<F>>().call(a...);
}

}  // namespace

TORCH_LIBRARY(paper_2408_11200_amd, m)
{
    m.def("kan_layer(Tensor x, Tensor coef, Tensor w_s, Tensor? w_b, int n_in, int n_out, int G, int k, float grid_lo, float grid_hi, "
          "int base_act) -> Tensor", &kan_layer);
    m.def("ukan_layer(Tensor x, Tensor E, Tensor W1, Tensor b1, Tensor W2, Tensor b2, Tensor scale, Tensor? w_b, int n_in, int n_out, "
          "int k, float h, int d_pe, int d_feat, int d_hidden, int base_act, int max_groups) -> Tensor", &ukan_layer);
}

PYBIND11_MODULE(_autograd, m)
{
    m.attr("torch_version") = KAN_TORCH_VERSION;    // of the torch the nodes are built on: autograd.py refuses another
    m.def("kan_layer", [](int32_t n_in, int32_t n_out, int32_t G, int32_t k, float lo, float hi, int32_t base_act, const Tensor &x,
                          const Tensor &coef, const Tensor &w_s, const std::optional<Tensor> &w_b) {
        return call(kKanOp, &kan_layer, x, coef, w_s, w_b, (int64_t)n_in, (int64_t)n_out, (int64_t)G, (int64_t)k, (double)lo, (double)hi,
                    (int64_t)base_act);
    });
    m.def("ukan_layer", [](int32_t n_in, int32_t n_out, int32_t k, float h, int32_t d_pe, int32_t d_feat, int32_t d_hidden, int32_t base_act,
                           int32_t max_groups, const Tensor &x, const Tensor &E, const Tensor &W1, const Tensor &b1, const Tensor &W2,
                           const Tensor &b2, const Tensor &scale, const std::optional<Tensor> &w_b) {
        return call(kUkanOp, &ukan_layer, x, E, W1, b1, W2, b2, scale, w_b, (int64_t)n_in, (int64_t)n_out, (int64_t)k, (double)h, (int64_t)d_pe,
                    (int64_t)d_feat, (int64_t)d_hidden, (int64_t)base_act, (int64_t)max_groups);
    });
}
