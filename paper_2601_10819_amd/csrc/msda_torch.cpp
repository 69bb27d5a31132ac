// The PyTorch side of the single-call operator in native code: argument
// checks, outputs, workspace and the C ABI call of forward and backward, and
// the autograd node.
//
// A small call is bound by the host, not by the GPU: with two cameras of 128 x
// 224 and 128 anchors the kernels of a forward take 7 us and those of a step
// 45 us, and enqueueing them from Python took 13.6 and 175 us -- most of the
// latter because the engine runs a Python node on a thread that has to wake
// up, take the interpreter lock and run cold. Here it is 5.0 and 69 us.
//
// The C ABI's functions are handed over by address (bind), so that the
// library called is the one the Python side has loaded.
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/custom_function.h>
#include <torch/csrc/autograd/functions/utils.h>
#include <torch/csrc/utils/pybind.h>
#include <torch/extension.h>

#include <array>
#include <mutex>
#include <string>
#include <vector>

#include "../../include/msda.h"

namespace py = pybind11;
using at::Tensor;
using c10::optional;

namespace {

// msda_forward_ws, msda_forward_workspace_size, msda_backward,
// msda_backward_workspace_size
struct Api {
    decltype(&msda_forward_ws) forward;
    decltype(&msda_forward_workspace_size) forward_bytes;
    decltype(&msda_backward) backward;
    decltype(&msda_backward_workspace_size) backward_bytes;
} g_api = {};

// What a call holds besides its feature, location and weight tensors. The
// host geometry is a copy: the caller may change or drop its own.
struct Call {
    Tensor shapes, starts;               // device geometry
    std::vector<int32_t> host_shapes, host_starts;
    int num_cams, num_levels;
    optional<Tensor> level_scale;
    bool deterministic, logits;
    bool has_tile;
    msda_tile tile;
};

std::string shape_text(at::IntArrayRef s) {
    std::string t = "(";
    for (size_t i = 0; i < s.size(); ++i)
        t += (i ? ", " : "") + std::to_string(s[i]);
    return t + (s.size() == 1 ? ",)" : ")");
}

std::string dtype_text(at::ScalarType t) {
    switch (t) {
        case at::kFloat: return "torch.float32";
        case at::kDouble: return "torch.float64";
        case at::kHalf: return "torch.float16";
        case at::kBFloat16: return "torch.bfloat16";
        case at::kInt: return "torch.int32";
        case at::kLong: return "torch.int64";
        default: return c10::toString(t);
    }
}

void need(const char* name, const Tensor& t, optional<at::ScalarType> dtype = {}) {
    if (!t.is_cuda()) throw py::value_error(std::string(name) + " must be a device tensor");
    if (!t.is_contiguous()) throw py::value_error(std::string(name) + " must be contiguous");
    if (dtype && t.scalar_type() != *dtype)
        throw py::value_error(std::string(name) + " must be " + dtype_text(*dtype) + ", got " +
                              dtype_text(t.scalar_type()));
}

void need_operands(const Tensor& feat, const Tensor& loc, const Tensor& w) {
    need("feat", feat);
    need("sampling_loc", loc, at::kFloat);
    need("weights", w);
    if (w.scalar_type() != at::kFloat && w.scalar_type() != at::kBFloat16)
        throw py::value_error("weights must be float32 or bfloat16, got " +
                              dtype_text(w.scalar_type()));
}

msda_desc make_desc(const Call& c, const Tensor& feat, const Tensor& loc, const Tensor& w) {
    if (feat.dim() != 3 || loc.dim() != 5 || w.dim() != 6)
        throw py::value_error(
            "feat [B,R,C], sampling_loc [B,A,P,Ncam,2], weights [B,A,P,Ncam,L,G]");
    const auto l = loc.sizes(), s = w.sizes();
    if (l[4] != 2 || l[0] != feat.size(0) || l[3] != c.num_cams)
        throw py::value_error("sampling_loc shape " + shape_text(l) + " does not match");
    if (s[0] != l[0] || s[1] != l[1] || s[2] != l[2] || s[3] != l[3] || s[4] != c.num_levels)
        throw py::value_error("weights shape " + shape_text(s) + " does not match");
    msda_desc d = {};
    switch (feat.scalar_type()) {
        case at::kFloat: d.feat_dtype = MSDA_F32; break;
        case at::kBFloat16: d.feat_dtype = MSDA_BF16; break;
        case at::kHalf: d.feat_dtype = MSDA_F16; break;
        case at::kByte:
        case at::kFloat8_e4m3fn: d.feat_dtype = MSDA_FP8_E4M3; break;
        default:
            throw py::value_error("unsupported feat dtype " + dtype_text(feat.scalar_type()));
    }
    d.batch = (int32_t)feat.size(0);
    d.num_cams = c.num_cams;
    d.num_levels = c.num_levels;
    d.num_anchors = (int32_t)l[1];
    d.num_points = (int32_t)l[2];
    d.channels = (int32_t)feat.size(2);
    d.groups = (int32_t)s[5];
    d.rows = feat.size(1);
    d.host_spatial_shapes = c.host_shapes.data();
    d.host_level_start_index = c.host_starts.data();
    d.level_scale = c.level_scale ? static_cast<const float*>(c.level_scale->data_ptr()) : nullptr;
    d.flags = (c.deterministic ? MSDA_DETERMINISTIC : 0) |
              (c.logits ? MSDA_WEIGHT_LOGITS : 0) |
              (w.scalar_type() == at::kBFloat16 ? MSDA_WEIGHTS_BF16 : 0);
    d.tile = c.has_tile ? &c.tile : nullptr;
    return d;
}

// A 256-byte aligned workspace of at least `bytes`: the caller's tensor if it
// is large enough, else a new one in *own.
struct Workspace {
    void* ptr = nullptr;
    size_t bytes = 0;
    Tensor own;

    Workspace(size_t need, const optional<Tensor>& given, const Tensor& like) {
        if (!need) return;
        if (given && use(*given) && bytes >= need) return;
        own = at::empty({(int64_t)need + 256}, like.options().dtype(at::kByte));
        use(own);
    }
    bool use(const Tensor& t) {
        const uintptr_t base = (uintptr_t)t.data_ptr(), at = (base + 255) / 256 * 256;
        const size_t size = (size_t)t.numel() * t.element_size();
        if (size < at - base) return false;
        ptr = (void*)at;
        bytes = size - (at - base);
        return true;
    }
};

void* current_stream() { return (void*)c10::hip::getCurrentHIPStream().stream(); }

msda_status run_forward(const Call& c, const Tensor& feat, const Tensor& loc, const Tensor& w,
                        const optional<Tensor>& workspace, void* stream, Tensor* out) {
    const msda_desc d = make_desc(c, feat, loc, w);
    if (!out->defined())
        *out = at::empty({d.batch, d.num_anchors, d.channels}, feat.options().dtype(at::kFloat));
    const Workspace ws(g_api.forward_bytes(&d), workspace, feat);
    return g_api.forward(feat.data_ptr(), (const int32_t*)c.shapes.data_ptr(),
                         (const int32_t*)c.starts.data_ptr(), (const float*)loc.data_ptr(),
                         (const float*)w.data_ptr(), (float*)out->data_ptr(), ws.ptr, ws.bytes, &d,
                         stream);
}

struct Grads {
    Tensor feat, loc, w;
};

msda_status run_backward(const Call& c, const Tensor& feat, const Tensor& loc, const Tensor& w,
                         const Tensor& grad_out, bool need_feat, bool need_loc, bool need_w,
                         const optional<Tensor>& workspace, void* stream, Grads* g) {
    need_operands(feat, loc, w);
    need("grad_out", grad_out, at::kFloat);
    const msda_desc d = make_desc(c, feat, loc, w);
    if (need_feat) g->feat = at::empty_like(feat);
    if (need_loc) g->loc = at::empty_like(loc);
    if (need_w) g->w = at::empty(w.sizes(), w.options().dtype(at::kFloat));
    auto ptr = [](const Tensor& t) { return t.defined() ? t.data_ptr() : nullptr; };
    const bool sized = need_feat || (d.flags & (MSDA_WEIGHT_LOGITS | MSDA_WEIGHTS_BF16));
    const Workspace ws(sized ? g_api.backward_bytes(&d) : 0, workspace, feat);
    return g_api.backward(feat.data_ptr(), (const int32_t*)c.shapes.data_ptr(),
                          (const int32_t*)c.starts.data_ptr(), (const float*)loc.data_ptr(),
                          (const float*)w.data_ptr(), (const float*)grad_out.data_ptr(),
                          ptr(g->feat), (float*)ptr(g->loc), (float*)ptr(g->w), ws.ptr, ws.bytes,
                          &d, stream);
}

// Raises the binding's MSDAError (with the interpreter lock).
void check(msda_status st) {
    if (st != MSDA_OK)
        py::module_::import("paper_2601_10819_amd._lib").attr("check")((int)st);
}

std::vector<int32_t> host_ints(const py::handle& a, size_t n) {
    Py_buffer b;
    if (PyObject_GetBuffer(a.ptr(), &b, PyBUF_C_CONTIGUOUS)) throw py::error_already_set();
    std::vector<int32_t> v;
    const bool fits = b.itemsize == 4 && (size_t)b.len == n * 4;
    if (fits) v.assign(static_cast<int32_t*>(b.buf), static_cast<int32_t*>(b.buf) + n);
    PyBuffer_Release(&b);
    if (!fits) throw py::value_error("host geometry: int32, one entry per camera and level");
    return v;
}

// tile: None or (waves_per_anchor, chans_per_lane, order, scatter).
void set_tile(Call* c, const py::handle& tile) {
    c->has_tile = !tile.is_none();
    c->tile = msda_tile{};
    if (c->has_tile) {
        const auto t = tile.cast<std::array<int32_t, 4>>();
        c->tile.waves_per_anchor = t[0];
        c->tile.chans_per_lane = t[1];
        c->tile.order = t[2];
        c->tile.scatter = t[3];
    }
}

// layout: ops.Layout.
Call make_call(const py::handle& layout, optional<Tensor> level_scale, bool deterministic,
               bool logits, const py::handle& tile) {
    Call c;
    c.num_cams = layout.attr("num_cams").cast<int>();
    c.num_levels = layout.attr("num_levels").cast<int>();
    const size_t n = (size_t)c.num_cams * (size_t)c.num_levels;
    c.host_shapes = host_ints(layout.attr("host_shapes"), 2 * n);
    c.host_starts = host_ints(layout.attr("host_starts"), n);
    c.shapes = layout.attr("shapes").cast<Tensor>();
    c.starts = layout.attr("starts").cast<Tensor>();
    c.level_scale = std::move(level_scale);
    c.deterministic = deterministic;
    c.logits = logits;
    set_tile(&c, tile);
    return c;
}

// f() without the interpreter lock: allocating and enqueueing can wait for the
// device, and other Python threads need not.
template <class F>
auto unlocked(F&& f) {
    py::gil_scoped_release free;
    return f();
}

void* stream_or_current(optional<int64_t> s) { return s ? (void*)*s : current_stream(); }

Tensor py_forward(const Tensor& feat, const py::handle& layout, const Tensor& loc, const Tensor& w,
                  optional<Tensor> level_scale, const py::handle& tile, optional<Tensor> out,
                  optional<Tensor> workspace, optional<int64_t> stream, bool logits) {
    need_operands(feat, loc, w);
    if (level_scale) need("level_scale", *level_scale, at::kFloat);
    const Call c = make_call(layout, std::move(level_scale), false, logits, tile);
    Tensor result = out ? *out : Tensor();
    check(unlocked([&] {
        return run_forward(c, feat, loc, w, workspace, stream_or_current(stream), &result);
    }));
    return result;
}

py::tuple py_backward(const Tensor& feat, const py::handle& layout, const Tensor& loc,
                      const Tensor& w, const Tensor& grad_out, bool need_feat, bool need_loc,
                      bool need_w, bool deterministic, const py::handle& tile,
                      optional<Tensor> workspace, optional<Tensor> level_scale,
                      optional<int64_t> stream, bool logits) {
    const Call c = make_call(layout, std::move(level_scale), deterministic, logits, tile);
    Grads g;
    check(unlocked([&] {
        return run_backward(c, feat, loc, w, grad_out, need_feat, need_loc, need_w, workspace,
                            stream_or_current(stream), &g);
    }));
    auto or_none = [](const Tensor& t) { return t.defined() ? py::cast(t) : py::none(); };
    return py::make_tuple(or_none(g.feat), or_none(g.loc), or_none(g.w));
}

// Raised on an engine's thread, which holds no interpreter lock: the Python
// error is set under it and travels with the exception.
[[noreturn]] void raise_python(msda_status st, const std::string& bad) {
    py::gil_scoped_acquire lock;
    if (!bad.empty()) {
        PyErr_SetString(PyExc_ValueError, bad.c_str());
    } else {
        try {
            check(st);
        } catch (py::error_already_set& e) {
            e.restore();
        }
    }
    python_error e;
    e.persist();
    throw e;
}

torch::autograd::variable_list call_backward(const Call& c, const Tensor& feat, const Tensor& loc,
                                             const Tensor& w, const Tensor& grad_out,
                                             bool need_feat, bool need_loc, bool need_w) {
    Grads g;
    if (need_feat || need_loc || need_w) {
        std::string bad;
        msda_status st = MSDA_OK;
        try {
            st = run_backward(c, feat, loc, w, grad_out.contiguous(), need_feat, need_loc, need_w,
                              {}, current_stream(), &g);
        } catch (const py::builtin_exception& e) {
            bad = e.what();
        }
        if (st != MSDA_OK || !bad.empty()) raise_python(st, bad);
        if (g.w.defined() && g.w.scalar_type() != w.scalar_type()) g.w = g.w.to(w.scalar_type());
    }
    return {g.feat, g.loc, g.w};
}

// The backward as compiled autograd calls it from its graph: the call's
// description taken from the node's saved data, where save put it.
struct MsdaBackward : torch::autograd::Function<MsdaBackward> {
    static void save(const Call& c, torch::autograd::AutogradContext* ctx) {
        std::vector<int64_t> v = {c.num_cams, c.num_levels, c.deterministic, c.logits, c.has_tile,
                                  c.tile.waves_per_anchor, c.tile.chans_per_lane, c.tile.order,
                                  c.tile.scatter};
        v.insert(v.end(), c.host_shapes.begin(), c.host_shapes.end());
        v.insert(v.end(), c.host_starts.begin(), c.host_starts.end());
        ctx->saved_data["call"] = std::move(v);
        ctx->saved_data["shapes"] = c.shapes;
        ctx->saved_data["starts"] = c.starts;
        if (c.level_scale) ctx->saved_data["level_scale"] = *c.level_scale;
    }

    static Call saved(torch::autograd::AutogradContext* ctx) {
        const auto v = ctx->saved_data["call"].toIntVector();
        Call c;
        c.num_cams = (int)v[0];
        c.num_levels = (int)v[1];
        c.deterministic = v[2];
        c.logits = v[3];
        c.has_tile = v[4];
        c.tile = msda_tile{};
        c.tile.waves_per_anchor = (int32_t)v[5];
        c.tile.chans_per_lane = (int32_t)v[6];
        c.tile.order = (int32_t)v[7];
        c.tile.scatter = (int32_t)v[8];
        const auto host = v.begin() + 9;
        const size_t n = (size_t)c.num_cams * (size_t)c.num_levels;
        c.host_shapes.assign(host, host + 2 * n);
        c.host_starts.assign(host + 2 * n, v.end());
        c.shapes = ctx->saved_data["shapes"].toTensor();
        c.starts = ctx->saved_data["starts"].toTensor();
        const auto scale = ctx->saved_data.find("level_scale");
        if (scale != ctx->saved_data.end()) c.level_scale = scale->second.toTensor();
        return c;
    }

    static torch::autograd::variable_list backward(torch::autograd::AutogradContext* ctx,
                                                   torch::autograd::variable_list grads) {
        const auto t = ctx->get_saved_variables();
        return call_backward(saved(ctx), t[0], t[1], t[2], grads[0], ctx->needs_input_grad(0),
                             ctx->needs_input_grad(1), ctx->needs_input_grad(2));
    }
};

// The autograd node of one call: torch's node of a C++ function (saved-tensor
// hooks, version checks, compiled autograd), the call's description beside it.
// The plain engine's pass reads that; it becomes saved data (a table of boxed
// values) only for compiled autograd, which takes the node apart: filling and
// reading the table on every call took 4.5 of a small step's 72 us.
struct MsdaNode : torch::autograd::CppNode<MsdaBackward> {
    Call call;

    std::string name() const override { return "MSDABackward"; }

    torch::autograd::variable_list apply(torch::autograd::variable_list&& grads) override {
        std::lock_guard<std::mutex> lock(mutex_);      // as release_variables takes it
        const auto t = ctx_.get_saved_variables();
        const Tensor go = grads[0].defined()
                              ? grads[0]
                              : at::zeros({t[1].size(0), t[1].size(1), t[0].size(2)},
                                          t[1].options());
        return call_backward(call, t[0], t[1], t[2], go, should_compute_output(0),
                             should_compute_output(1), should_compute_output(2));
    }

    void compiled_args(torch::dynamo::autograd::CompiledNodeArgs& args) const override {
        MsdaBackward::save(call, const_cast<torch::autograd::AutogradContext*>(&ctx_));
        CppNode::compiled_args(args);
    }
};

Tensor py_msda(const Tensor& feat, const py::handle& layout, const Tensor& loc, const Tensor& w,
               optional<Tensor> level_scale, bool deterministic, const py::handle& tile_forward,
               const py::handle& tile_backward, bool logits) {
    need_operands(feat, loc, w);
    if (level_scale) need("level_scale", *level_scale, at::kFloat);
    Call c = make_call(layout, std::move(level_scale), deterministic, logits, tile_forward);
    Tensor out;
    c.deterministic = false;                    // the forward knows no such flag
    check(unlocked([&] { return run_forward(c, feat, loc, w, {}, current_stream(), &out); }));
    if (torch::autograd::compute_requires_grad(feat, loc, w)) {
        auto node = std::shared_ptr<MsdaNode>(new MsdaNode(), torch::autograd::deleteNode);
        node->set_next_edges(torch::autograd::collect_next_edges(feat, loc, w));
        node->set_ctx_grad_fn(node);
        c.deterministic = deterministic;
        set_tile(&c, tile_backward);
        node->call = std::move(c);
        node->ctx_.save_for_backward({feat, loc, w});
        node->is_variable_input_ = {true, true, true};
        for (const Tensor& t : {feat, loc, w}) node->input_info_.emplace_back(t);
        torch::autograd::set_history(out, node);
        node->output_info_.emplace_back(out);
        node->save_variables_to_ctx();
    }
    return out;
}

void bind(uintptr_t forward, uintptr_t forward_bytes, uintptr_t backward,
          uintptr_t backward_bytes) {
    g_api.forward = reinterpret_cast<decltype(g_api.forward)>(forward);
    g_api.forward_bytes = reinterpret_cast<decltype(g_api.forward_bytes)>(forward_bytes);
    g_api.backward = reinterpret_cast<decltype(g_api.backward)>(backward);
    g_api.backward_bytes = reinterpret_cast<decltype(g_api.backward_bytes)>(backward_bytes);
}

}  // namespace

PYBIND11_MODULE(_msda_torch, m) {
    m.def("bind", &bind);
    // (out of memory and the like become torch's own Python errors)
    m.def("forward", torch::wrap_pybind_function(py_forward));
    m.def("backward", torch::wrap_pybind_function(py_backward));
    m.def("msda", torch::wrap_pybind_function(py_msda));
}
