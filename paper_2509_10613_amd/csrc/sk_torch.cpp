// The autograd wrappers' host path in native code: the same calls of the C ABI, with the same arguments, as the
// torch.autograd.Function classes in autograd.py, as nodes of PyTorch's own graph.
//
// What it is for: a training pass over a few short paths is bound by the host.  8 pairs of 16 points, forward and backward
// through the Python classes: 66 us where one core runs both threads, 143 us where the autograd engine's thread runs on
// another one, which then goes through the interpreter, ctypes and the argument checks with cold caches; a Python class that
// does nothing takes 24 and 53 us.  What the calls launch is not changed.
//
// Every function returns None for a call that it leaves to the Python classes: anything but plain device tensors of one
// floating type and consistent shapes and int arguments, calls under a tracer or a function transform, kept workspaces
// above the given limit (their accounting lives there), and whatever the library refuses (the classes then raise).
#include <ATen/ATen.h>
#include <ATen/SavedTensorHooks.h>
#include <c10/core/impl/LocalDispatchKeySet.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/custom_function.h>
#include <torch/csrc/autograd/edge.h>
#include <torch/csrc/autograd/function.h>
#include <torch/csrc/autograd/functions/utils.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/autograd/saved_variable.h>
#include <torch/csrc/autograd/variable.h>
#include <torch/csrc/jit/frontend/tracer.h>
#include <torch/csrc/utils/pybind.h>

#include <array>
#include <atomic>
#include <cstring>
#include <limits>
#include <memory>
#include <mutex>
#include <string>

#include "sigkernel.h"
#include "signature.h"

namespace {

using at::Tensor;
using torch::autograd::Node;
using torch::autograd::SavedVariable;
using torch::autograd::variable_list;

void* current_stream() { return static_cast<void*>(c10::hip::getCurrentHIPStream().stream()); }
sk_dtype dtype_of(const Tensor& t) { return t.scalar_type() == at::kDouble ? SK_F64 : SK_F32; }
Tensor bytes(size_t n, const Tensor& like) { return at::empty({(int64_t)(n < 256 ? 256 : n)}, like.options().dtype(at::kByte)); }
// The workspace a call is fastest with or, where the device has no room for it, half of that and so on down to the least the
// call takes.
template <class F>
Tensor workspace(size_t n, const Tensor& like, F&& least)
{
    for (size_t few = 0;;) {
        try {
            return bytes(n, like);
        } catch (const c10::OutOfMemoryError&) {
            if (few == 0) few = least();
            if (n <= few) throw;
        }
        n = n / 2 > few ? n / 2 : few;
    }
}
void* ptr(const Tensor& t) { return t.defined() ? t.data_ptr() : nullptr; }

// (the exception that the classes raise)
void check(int rc)
{
    if (rc == SK_OK) return;
    const std::string what = "sigkernel error " + std::to_string(rc) + ": " + sigkernel_last_error();
    py::gil_scoped_acquire gil;
    PyErr_SetString(py::module_::import("paper_2509_10613_amd.binding").attr("SigKernelError").ptr(), what.c_str());
    python_error error;
    error.persist();   // (it crosses from the engine's thread to the caller's)
    throw error;
}

// ---------------------------------------------------------------- what a shape needs
// Workspace sizes and whether the forward sweep is kept, by shape and flags: arithmetic on the host that the library would
// repeat in every call.  The last few shapes of each thread.
struct Need {
    size_t forward, kept, backward;   // kept: the forward call that keeps what it sweeps (0: the shape has no such form)
    int keep, have;                   // the flags of that form, forward and backward
};
struct ShapeKey {
    int64_t v[8];
};
template <class F>
const Need& need_of(const ShapeKey& key, F&& compute)
{
    constexpr int kPlaces = 32;
    static thread_local std::array<ShapeKey, kPlaces> keys{};
    static thread_local std::array<Need, kPlaces> needs{};
    static thread_local int filled = 0, next = 0;
    for (int i = 0; i < filled; ++i)
        if (std::memcmp(&keys[i], &key, sizeof(key)) == 0) return needs[i];
    const int at = next;
    next = (next + 1) % kPlaces;
    needs[at] = compute();
    keys[at] = key;
    if (at >= filled) filled = at + 1;
    return needs[at];
}

Need kernel_need(bool gram, bool symmetric, int64_t N, int64_t M, int64_t L1, int64_t L2, int64_t d, int lam1, int lam2, int flags,
                 sk_dtype dt)
{
    const int fwd = gram ? SK_OP_GRAM : SK_OP_FWD, bwd = gram ? SK_OP_GRAM_BWD : SK_OP_BWD;
    auto size = [&](int op, int f) { return sigkernel_workspace_bytes(op, N, M, L1, L2, d, lam1, lam2, f, dt); };
    Need n{size(fwd, flags), 0, size(bwd, flags), SK_FLAG_KEEP_FORWARD, SK_FLAG_HAVE_FORWARD};
    if (N < 1 || L1 < 2 || L2 < 2 || (gram && M < 1)) return n;
    char text[1024];
    if (sigkernel_describe(fwd, N, M, L1, L2, d, lam1, lam2, flags | SK_FLAG_KEEP_SWEEPS, dt, text, sizeof(text)) == SK_OK &&
        std::strstr(text, " kept_sweeps=2")) {
        n.keep = SK_FLAG_KEEP_SWEEPS;
        n.have = SK_FLAG_HAVE_SWEEPS;
        n.kept = size(fwd, flags | SK_FLAG_KEEP_SWEEPS);
        return n;
    }
    if (sigkernel_describe(fwd, N, M, L1, L2, d, lam1, lam2, flags | SK_FLAG_KEEP_FORWARD, dt, text, sizeof(text)) != SK_OK ||
        !std::strstr(text, " kept_sweep_half=1 "))
        return n;
    // (the backward sweep with four pairs per wavefront makes its own forward sweep, and is mostly faster than the kept form)
    if (gram) {
        if (sigkernel_describe(bwd, N, M, L1, L2, d, lam1, lam2, flags, dt, text, sizeof(text)) != SK_OK) return n;
        if (std::strstr(text, symmetric ? " symmetric_over_kept_sweep=1" : " over_kept_sweep=1")) return n;
    }
    n.kept = size(fwd, flags | SK_FLAG_KEEP_FORWARD);
    return n;
}

// ---------------------------------------------------------------- graph nodes
// A backward call's tensor (what a saved-tensor hook gave back, an upstream gradient) as the forward call knew it: the library
// takes addresses.
void expect(const Tensor& t, const char* name, at::IntArrayRef sizes, const at::TensorOptions& options)
{
    TORCH_CHECK_VALUE(t.is_cuda() && t.layout() == at::kStrided && t.is_contiguous(), name, " must be a contiguous device tensor");
    TORCH_CHECK_VALUE(t.device() == options.device() && t.scalar_type() == c10::typeMetaToScalarType(options.dtype()) && t.sizes() == sizes,
                      name, " is not what the forward call had: ", t.sizes(), " ", t.scalar_type(), " on ", t.device());
}

// Bytes of kept sweeps that the live graphs hold on a device: a share of it, given back with the graph.
class Share {
public:
    // false: all shares would come to more than `most`
    bool take(const Tensor& like, size_t bytes, size_t most)
    {
        static std::array<std::atomic<int64_t>, 64> held;
        auto& all = held[(size_t)like.device().index() % held.size()];
        if (all.fetch_add((int64_t)bytes) + (int64_t)bytes > (int64_t)most) {
            all.fetch_sub((int64_t)bytes);
            return false;
        }
        all_ = &all;
        bytes_ = (int64_t)bytes;
        return true;
    }
    void give_back()
    {
        if (all_) all_->fetch_sub(bytes_);
        all_ = nullptr;
    }
    Share() = default;
    Share(Share&& o) noexcept : all_(o.all_), bytes_(o.bytes_) { o.all_ = nullptr; }
    Share& operator=(Share&& o) noexcept
    {
        give_back();
        all_ = o.all_;
        bytes_ = o.bytes_;
        o.all_ = nullptr;
        return *this;
    }
    ~Share() { give_back(); }

private:
    std::atomic<int64_t>* all_ = nullptr;
    int64_t bytes_ = 0;
};

// (Threads may run backward calls through one node: what it holds is read and released under the node's lock.)
using Lock = std::lock_guard<std::mutex>;

struct KernelNode : public Node {
    SavedVariable x_, y_;
    bool gram = false, symmetric = false, want_x = false, want_y = false;
    int lam1 = 0, lam2 = 0, flags = 0, have = 0;
    size_t need = 0;
    Tensor ws;                       // the kept sweeps
    Share share;                     // ... and what of all kept sweeps they are
    const void *x_at = nullptr, *y_at = nullptr;   // the paths they belong to
    std::vector<int64_t> x_sizes, y_sizes, out_sizes;
    at::TensorOptions options;

    std::string name() const override { return gram ? "SigKernelGramBackward" : "SigKernelPairBackward"; }
    void release_variables() override
    {
        const Lock lock(mutex_);
        x_.reset_data();
        y_.reset_data();
        ws.reset();
        share.give_back();
    }
    variable_list apply(variable_list&& grads) override
    {
        variable_list out(symmetric ? 1 : 2);
        if (!want_x && !want_y) return out;
        Tensor x, y, held;
        {
            const Lock lock(mutex_);
            x = x_.unpack();
            y = symmetric ? x : y_.unpack();
            held = ws;
        }
        const Tensor g = grads[0].defined() ? grads[0].contiguous() : at::zeros(out_sizes, options);
        expect(x, "x", x_sizes, options);
        if (!symmetric) expect(y, "y", y_sizes, options);
        expect(g, "the upstream gradient", out_sizes, options);
        // (paths whose data have been set elsewhere are another call's to the library)
        const bool kept = held.defined() && x.data_ptr() == x_at && y.data_ptr() == y_at;
        const int f = flags | (kept ? have : 0);
        const sk_dtype dt = dtype_of(x);
        const int64_t N = x.size(0), M = y.size(0), L1 = x.size(1), L2 = y.size(1), d = x.size(2);
        const Tensor w = kept ? held : workspace(need, x, [&] {
            return sigkernel_workspace_least_bytes(gram ? SK_OP_GRAM_BWD : SK_OP_BWD, N, M, L1, L2, d, lam1, lam2, f, dt);
        });
        // (a Gram call computes both sides)
        Tensor gx, gy;
        if (want_x || gram) gx = at::empty_like(x, at::MemoryFormat::Contiguous);
        if ((want_y || gram) && !symmetric) gy = at::empty_like(y, at::MemoryFormat::Contiguous);
        const Tensor k = at::empty(out_sizes, options);
        if (gram)
            check(sigkernel_gram(x.data_ptr(), y.data_ptr(), k.data_ptr(), g.data_ptr(), ptr(gx), ptr(gy), N, M, L1, L2, d, lam1, lam2, f,
                                 dt, w.data_ptr(), (size_t)w.numel(), current_stream()));
        else
            check(sigkernel_bwd(x.data_ptr(), y.data_ptr(), g.data_ptr(), ptr(gx), ptr(gy), k.data_ptr(), N, L1, L2, d, lam1, lam2, f, dt,
                                w.data_ptr(), (size_t)w.numel(), current_stream()));
        if (want_x) out[0] = gx;
        if (want_y && !symmetric) out[1] = gy;
        return out;
    }
};

// The gradients are the forward call's, and the backward call is tensor arithmetic: a function of PyTorch's own kind, whose
// nodes compiled autograd takes as well.
struct MmdParts {
    Tensor loss, gx, gy;   // gx, gy: undefined where not wanted
};
struct SigMmd2 : public torch::autograd::Function<SigMmd2> {
    static Tensor forward(torch::autograd::AutogradContext* ctx, const Tensor&, const Tensor&, const MmdParts& parts)
    {
        variable_list grads;
        for (const Tensor& g : {parts.gx, parts.gy})
            if (g.defined()) grads.push_back(g);
        ctx->save_for_backward(grads);
        ctx->saved_data["have_x"] = parts.gx.defined();
        ctx->saved_data["have_y"] = parts.gy.defined();
        return parts.loss;
    }
    static variable_list backward(torch::autograd::AutogradContext* ctx, const variable_list& grads)
    {
        variable_list out(3);
        const variable_list saved = ctx->get_saved_variables();
        const bool have_x = ctx->saved_data["have_x"].toBool(), have_y = ctx->saved_data["have_y"].toBool();
        if (have_x) out[0] = saved[0] * grads[0];
        if (have_y) out[1] = saved[have_x ? 1 : 0] * grads[0];
        return out;
    }
};

struct SignatureNode : public Node {
    SavedVariable x_, out_;
    int N = 0, flags = 0;
    size_t need = 0;
    std::vector<int64_t> x_sizes, out_sizes;
    at::TensorOptions options;
    std::string name() const override { return "SignatureBackward"; }
    void release_variables() override
    {
        const Lock lock(mutex_);
        x_.reset_data();
        out_.reset_data();
    }
    variable_list apply(variable_list&& grads) override
    {
        Tensor x, sig;
        {
            const Lock lock(mutex_);
            x = x_.unpack();
            sig = out_.unpack(shared_from_this());
        }
        const Tensor g = grads[0].defined() ? grads[0].contiguous() : at::zeros(out_sizes, options);
        expect(x, "x", x_sizes, options);
        expect(sig, "the signatures", out_sizes, options);
        expect(g, "the upstream gradient", out_sizes, options);
        const Tensor gx = at::empty_like(x, at::MemoryFormat::Contiguous);
        const Tensor w = bytes(need, x);
        check(signature_bwd(x.data_ptr(), sig.data_ptr(), g.data_ptr(), gx.data_ptr(), x.size(0), x.size(1), x.size(2), N, flags,
                            dtype_of(x), w.data_ptr(), (size_t)w.numel(), current_stream()));
        return {gx};
    }
};

template <class T>
std::shared_ptr<T> make_node()
{
    return std::shared_ptr<T>(new T(), torch::autograd::deleteNode);
}

// ---------------------------------------------------------------- which calls are taken
bool transformed()
{
    return c10::impl::tls_is_dispatch_key_included(c10::DispatchKey::FuncTorchDynamicLayerFrontMode) ||
           c10::impl::tls_is_dispatch_key_included(c10::DispatchKey::Python) || torch::jit::tracer::isTracing();
}
// a three-dimensional device tensor of a type the library takes, without forward gradients
bool plain(const py::object& o, Tensor& t)
{
    if (!THPVariable_Check(o.ptr())) return false;
    t = THPVariable_Unpack(o.ptr());
    return t.is_cuda() && t.dim() == 3 && t.layout() == at::kStrided && (t.scalar_type() == at::kDouble || t.scalar_type() == at::kFloat) &&
           !t.key_set().has(c10::DispatchKey::Python) && !t._fw_grad(0).defined();
}
bool number(const py::object& o, int& v)
{
    if (!PyLong_Check(o.ptr())) return false;
    int overflow = 0;
    const long long l = PyLong_AsLongLongAndOverflow(o.ptr(), &overflow);
    if (overflow || l < INT32_MIN || l > INT32_MAX) return false;
    v = (int)l;
    return true;
}

// flags of the wrappers (those that keep a forward sweep or take one over are theirs to set)
bool flag_bits(const py::object& o, int& v) { return number(o, v) && (v & (SK_FLAG_KEEP_FORWARD | SK_FLAG_HAVE_FORWARD | SK_FLAG_KEEP_SWEEPS | SK_FLAG_HAVE_SWEEPS)) == 0; }

// Whether what a call saves goes through hooks.  Its backward call may then get anything back, recomputed or rounded, at any
// address, and what the forward call would keep would mostly lie there unused: a checkpointed segment is run again.
bool saving_through_hooks() { return at::SavedTensorDefaultHooks::get_hooks().has_value(); }

// ---------------------------------------------------------------- the calls
Tensor kernel_call(const Tensor& x0, const Tensor& y0, bool gram, bool symmetric, int lam1, int lam2, int flags, size_t keep_limit,
                   size_t keep_all)
{
    const bool grad = at::GradMode::is_enabled() && (x0.requires_grad() || y0.requires_grad());
    Tensor x, y, k, ws;
    size_t need_bwd;
    int have = 0;
    bool kept = false;
    Share share;
    {
        at::NoGradGuard no_grad;
        x = x0.contiguous();
        y = symmetric ? x : y0.contiguous();
        const sk_dtype dt = dtype_of(x);
        const int64_t N = x.size(0), M = y.size(0), L1 = x.size(1), L2 = y.size(1), d = x.size(2);
        const ShapeKey key{{(int64_t)gram | (int64_t)symmetric << 1 | (int64_t)dt << 2, N, M, L1, L2, d, (int64_t)lam1 << 32 | (uint32_t)lam2,
                            flags}};
        const Need need = need_of(key, [&] { return kernel_need(gram, symmetric, N, gram ? M : 0, L1, L2, d, lam1, lam2, flags, dt); });
        const bool keep = grad && need.kept != 0 && !saving_through_hooks();
        if (keep && need.kept > keep_limit) return {};
        need_bwd = need.backward;
        have = need.have;
        if (keep && share.take(x, need.kept, keep_all)) {
            try {
                ws = bytes(need.kept, x);
                kept = true;
            } catch (const c10::OutOfMemoryError&) {   // the calls go on without one
                share.give_back();
            }
        }
        if (!kept)
            ws = workspace(need.forward, x, [&] {
                return sigkernel_workspace_least_bytes(gram ? SK_OP_GRAM : SK_OP_FWD, N, M, L1, L2, d, lam1, lam2, flags, dt);
            });
        const int f = flags | (kept ? need.keep : 0);
        int rc;
        if (gram) {
            k = at::empty({N, M}, x.options());
            rc = sigkernel_gram(x.data_ptr(), y.data_ptr(), k.data_ptr(), nullptr, nullptr, nullptr, N, M, L1, L2, d, lam1, lam2, f, dt,
                                ws.data_ptr(), (size_t)ws.numel(), current_stream());
        } else {
            k = at::empty({N}, x.options());
            rc = sigkernel_fwd(x.data_ptr(), y.data_ptr(), k.data_ptr(), N, L1, L2, d, lam1, lam2, f, dt, ws.data_ptr(),
                               (size_t)ws.numel(), current_stream());
        }
        if (rc != SK_OK) return {};
    }
    if (grad) {
        auto node = make_node<KernelNode>();
        if (symmetric) node->set_next_edges(torch::autograd::collect_next_edges(x0));
        else node->set_next_edges(torch::autograd::collect_next_edges(x0, y0));
        node->x_ = SavedVariable(x, false);
        if (!symmetric) node->y_ = SavedVariable(y, false);
        node->gram = gram;
        node->symmetric = symmetric;
        node->want_x = x0.requires_grad();
        node->want_y = !symmetric && y0.requires_grad();
        node->lam1 = lam1;
        node->lam2 = lam2;
        node->flags = flags;
        node->have = have;
        node->need = need_bwd;
        if (kept) {
            node->ws = ws;
            node->share = std::move(share);
        }
        node->x_at = x.data_ptr();
        node->y_at = y.data_ptr();
        node->x_sizes = x.sizes().vec();
        node->y_sizes = y.sizes().vec();
        node->out_sizes = k.sizes().vec();
        node->options = k.options();
        torch::autograd::set_history(k, node);
    }
    return k;
}

py::object wrap(const Tensor& t)
{
    if (!t.defined()) return py::none();
    return py::reinterpret_steal<py::object>(THPVariable_Wrap(t));
}

py::object pair(py::object xo, py::object yo, py::object l1, py::object l2, py::object fl, size_t keep_limit, size_t keep_all)
{
    Tensor x, y, k;
    int lam1, lam2, flags;
    if (transformed() || !plain(xo, x) || !plain(yo, y) || !number(l1, lam1) || !number(l2, lam2) || !flag_bits(fl, flags) ||
        x.size(0) != y.size(0) || x.size(2) != y.size(2) || x.scalar_type() != y.scalar_type() || x.device() != y.device())
        return py::none();
    {
        py::gil_scoped_release release;
        k = kernel_call(x, y, false, false, lam1, lam2, flags, keep_limit, keep_all);
    }
    return wrap(k);
}

// Y None: K(X, X)
py::object gram(py::object xo, py::object yo, py::object l1, py::object l2, py::object fl, size_t keep_limit, size_t keep_all)
{
    Tensor x, y, k;
    int lam1, lam2, flags;
    const bool symmetric = yo.is_none();
    if (transformed() || !plain(xo, x) || !number(l1, lam1) || !number(l2, lam2) || !flag_bits(fl, flags)) return py::none();
    if (symmetric) y = x;
    else if (!plain(yo, y) || x.size(2) != y.size(2) || x.scalar_type() != y.scalar_type() || x.device() != y.device())
        return py::none();
    // (the library takes one address on both sides for K(X, X))
    if (!symmetric && x.data_ptr() == y.data_ptr()) return py::none();
    {
        py::gil_scoped_release release;
        k = kernel_call(x, y, true, symmetric, lam1, lam2, flags, keep_limit, keep_all);
    }
    return wrap(k);
}

py::object mmd2(py::object xo, py::object yo, py::object l1, py::object l2, py::object fl)
{
    Tensor x0, y0, loss;
    int lam1, lam2, flags;
    if (transformed() || !plain(xo, x0) || !plain(yo, y0) || !number(l1, lam1) || !number(l2, lam2) || !flag_bits(fl, flags) ||
        x0.size(2) != y0.size(2) || x0.scalar_type() != y0.scalar_type() || x0.device() != y0.device())
        return py::none();
    {
        py::gil_scoped_release release;
        const bool grad = at::GradMode::is_enabled();
        const bool want_x = grad && x0.requires_grad(), want_y = grad && y0.requires_grad();
        Tensor gx, gy;
        {
            at::NoGradGuard no_grad;
            const Tensor x = x0.contiguous(), y = y0.contiguous();
            const sk_dtype dt = dtype_of(x);
            const int64_t N = x.size(0), M = y.size(0), L1 = x.size(1), L2 = y.size(1), d = x.size(2);
            const ShapeKey key{{8 | (int64_t)(want_x || want_y) << 1 | (int64_t)dt << 2, N, M, L1, L2, d, (int64_t)lam1 << 32 | (uint32_t)lam2, flags}};
            const Need need = need_of(key, [&] {
                return Need{sigkernel_mmd2_workspace_bytes(N, M, L1, L2, d, lam1, lam2, flags, dt, want_x || want_y ? 1 : 0), 0, 0, 0, 0};
            });
            loss = at::empty({}, x.options());
            if (want_x) gx = at::empty_like(x, at::MemoryFormat::Contiguous);
            if (want_y) gy = at::empty_like(y, at::MemoryFormat::Contiguous);
            const Tensor ws = workspace(need.forward, x, [&] {
                return sigkernel_mmd2_workspace_least_bytes(N, M, L1, L2, d, lam1, lam2, flags, dt, want_x || want_y ? 1 : 0);
            });
            if (sigkernel_mmd2(x.data_ptr(), y.data_ptr(), loss.data_ptr(), ptr(gx), ptr(gy), N, M, L1, L2, d, lam1, lam2, flags, dt,
                               ws.data_ptr(), (size_t)ws.numel(), current_stream()) != SK_OK)
                loss.reset();
        }
        if (loss.defined() && (want_x || want_y)) loss = SigMmd2::apply(x0, y0, MmdParts{loss, gx, gy});
    }
    return wrap(loss);
}

py::object signature(py::object xo, py::object No, py::object fl)
{
    Tensor x0, out;
    int N, flags;
    if (transformed() || !plain(xo, x0) || !number(No, N) || !number(fl, flags)) return py::none();
    {
        py::gil_scoped_release release;
        const bool grad = at::GradMode::is_enabled() && x0.requires_grad();
        const int64_t B = x0.size(0), L = x0.size(1), d = x0.size(2), n = signature_length(d, N, flags);
        const sk_dtype dt = dtype_of(x0);
        Tensor x;
        Need need{};
        if (n > 0) {
            at::NoGradGuard no_grad;
            x = x0.contiguous();
            const ShapeKey key{{16 | (int64_t)dt << 2, B, 0, L, 0, d, N, flags}};
            need = need_of(key, [&] {
                return Need{signature_workspace_bytes(B, L, d, N, flags, dt), 0, signature_bwd_workspace_bytes(B, L, d, N, flags, dt, 1), 0, 0};
            });
            out = at::empty({B, n}, x.options());
            const Tensor ws = bytes(need.forward, x);
            if (signature_fwd(x.data_ptr(), out.data_ptr(), B, L, d, N, flags, dt, ws.data_ptr(), (size_t)ws.numel(), current_stream()) != SK_OK)
                out.reset();
        }
        if (out.defined() && grad) {
            auto node = make_node<SignatureNode>();
            node->set_next_edges(torch::autograd::collect_next_edges(x0));
            node->x_ = SavedVariable(x, false);
            node->N = N;
            node->flags = flags;
            node->need = need.backward;
            node->x_sizes = x.sizes().vec();
            node->out_sizes = out.sizes().vec();
            node->options = out.options();
            torch::autograd::set_history(out, node);
            node->out_ = SavedVariable(out, true);
        }
    }
    return wrap(out);
}

// The rule for the classes: what a forward call of this shape keeps for its backward call, in bytes (0: nothing), and the flags
// of that form, forward and backward.
py::tuple kept_form(bool gram, bool symmetric, int64_t N, int64_t M, int64_t L1, int64_t L2, int64_t d, int lam1, int lam2, int flags,
                    int dt)
{
    const Need n = kernel_need(gram, symmetric, N, M, L1, L2, d, lam1, lam2, flags, (sk_dtype)dt);
    return py::make_tuple(n.kept, n.keep, n.have);
}

}  // namespace

PYBIND11_MODULE(_native, m)
{
    m.def("kept_form", &kept_form);
    m.def("saving_through_hooks", &saving_through_hooks);
    // keep_limit: bytes that one call may keep (more is the classes' business); keep_all: that all live graphs may, on a device
    const auto all = py::arg("keep_all") = std::numeric_limits<int64_t>::max();
    m.def("pair", &pair, py::arg("x"), py::arg("y"), py::arg("lam1"), py::arg("lam2"), py::arg("flags"), py::arg("keep_limit"), all);
    m.def("gram", &gram, py::arg("x"), py::arg("y"), py::arg("lam1"), py::arg("lam2"), py::arg("flags"), py::arg("keep_limit"), all);
    m.def("mmd2", &mmd2);
    m.def("signature", &signature);
}
