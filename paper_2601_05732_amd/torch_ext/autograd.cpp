// The graph nodes of paper_2601_05732_amd/autograd.py in C++: the same calls into libmhcl, the same tensors kept and
// the same gradients returned, without the interpreter between them.  A stack's host time is a graph node and a few
// allocations per library call: a step of two layers at n = 4, C = 1024, 2048 tokens, of which the kernels take 190 us, took 414 us
// with the nodes in Python; with these and the ends' own kernels 193 on the same inputs again and again, 270 on new ones.
//
// autograd.py decides which calls come here: plain GPU tensors outside of function transforms, tracing and
// dispatch modes, with every shape, type and layout checked.  What the library itself refuses is raised as its status.
#include <torch/extension.h>

#include <c10/hip/HIPStream.h>

#include <tuple>

#include "../../include/mhcl.h"

namespace {

using at::Tensor;
using torch::autograd::AutogradContext;
using torch::autograd::Function;
using torch::autograd::variable_list;

// Raises what binding.py raises for the same status. As a Python exception from here on: a backward runs in autograd's
// threads, which carry those over to the caller as they are and make a RuntimeError of all others.
[[noreturn]] void raise(int status, const char *where) {
  py::gil_scoped_acquire gil;
  const py::object type = py::module_::import("paper_2601_05732_amd.binding").attr("MhclError"), error = type(status, where);
  PyErr_SetObject(type.ptr(), error.ptr());
  python_error e;
  e.persist();
  throw e;
}
void check(int status, const char *where) {
  if (status != MHCL_OK) raise(status, where);
}

void *stream() { return c10::hip::getCurrentHIPStream().stream(); }

// an empty tensor has no storage: NULL
template <typename T = void>
T *ptr(const Tensor &t) {
  return t.numel() == 0 ? nullptr : static_cast<T *>(t.data_ptr());
}
Tensor floats(const Tensor &like, at::IntArrayRef shape) { return at::empty(shape, like.options().dtype(at::kFloat)); }

// as layer.empty_stream: contiguous, first byte `phase` bytes past a 1 KiB boundary
Tensor empty_stream(const Tensor &like, at::IntArrayRef shape, int64_t phase) {
  int64_t numel = 1;
  std::vector<int64_t> strides(shape.size());
  for (size_t i = shape.size(); i-- > 0;) {
    strides[i] = numel;
    numel *= shape[i];
  }
  const int64_t size = like.element_size();
  const Tensor buf = at::empty({numel + 1024 / size}, like.options());
  const uintptr_t lead = (static_cast<uintptr_t>(phase) - reinterpret_cast<uintptr_t>(buf.data_ptr())) & 1023u;
  return buf.as_strided(shape, strides, static_cast<int64_t>(lead) / size);
}

// What the nodes of a layer share: its description, and what the post node leaves for the coefficient node.
struct Link final : torch::CustomClassHolder {
  mhcl_desc d;
  Tensor perm;                      // keeps d.perm alive
  int64_t g_x_phase;
  Tensor y, g_xout;                 // (y without its history: with it the link would hold itself)
};
using LinkPtr = c10::intrusive_ptr<Link>;

c10::IValue keep(const LinkPtr &link) {
  return c10::IValue::make_capsule(c10::static_intrusive_pointer_cast<torch::CustomClassHolder>(link));
}
LinkPtr kept(AutogradContext *ctx) {
  return c10::static_intrusive_pointer_cast<Link>(ctx->saved_data["link"].toCapsule());
}

Tensor workspace(const mhcl_desc &d, int op, const Tensor &like) {
  return at::empty({static_cast<int64_t>(mhcl_workspace_bytes(&d, op))}, like.options().dtype(at::kByte));
}

struct CoeffsPre : Function<CoeffsPre> {
  static variable_list forward(AutogradContext *ctx, Tensor x, Tensor W, Tensor b, Tensor alpha, LinkPtr link) {
    const mhcl_desc &d = link->d;
    const Tensor H_res = floats(x, {d.T, d.n, d.n}), H_pre = floats(x, {d.T, d.n}), H_post = floats(x, {d.T, d.n});
    const Tensor h = at::empty({d.T, d.C}, x.options()), ws = workspace(d, MHCL_OP_FWD_COEFFS_PRE, x);
    check(mhcl_fwd_coeffs_pre(&d, ptr(x), ptr<float>(W), ptr<float>(b), ptr<float>(alpha), ptr<float>(H_res),
                              ptr<float>(H_pre), ptr<float>(H_post), ptr(h), ws.data_ptr(), ws.nbytes(), stream()),
          "mhcl_fwd_coeffs_pre");
    ctx->save_for_backward({x, W, b, alpha});
    ctx->saved_data["link"] = keep(link);
    ctx->mark_non_differentiable({H_pre});
    ctx->set_materialize_grads(false);   // the gradients on H_* are not read: no zeros for them
    return {h, H_res, H_post, H_pre};
  }

  static variable_list backward(AutogradContext *ctx, variable_list grads) {
    const variable_list saved = ctx->get_saved_variables();
    const Tensor &x = saved[0], &W = saved[1], &b = saved[2], &alpha = saved[3];
    const LinkPtr link = kept(ctx);
    const mhcl_desc &d = link->d;
    TORCH_CHECK(link->y.defined(), "hyper-connection backward: the post update of this layer was never run");
    const Tensor g_xout = link->g_xout.defined() ? link->g_xout : at::zeros_like(x);
    const Tensor g_h = grads[0].defined() ? grads[0].contiguous() : at::zeros({d.T, d.C}, x.options());
    const Tensor g_x = empty_stream(x, x.sizes(), link->g_x_phase);
    const Tensor g_W = floats(x, W.sizes()), g_b = floats(x, b.sizes()), g_alpha = floats(x, {3});
    const Tensor ws = workspace(d, MHCL_OP_BWD_FUSED, x);
    // g_y went out through the post node already: not asked for again
    check(mhcl_bwd_fused(&d, ptr(x), ptr(link->y), ptr<float>(W), ptr<float>(b), ptr<float>(alpha), ptr(g_xout), ptr(g_h),
                         ptr(g_x), nullptr, ptr<float>(g_W), ptr<float>(g_b), ptr<float>(g_alpha), ws.data_ptr(),
                         ws.nbytes(), stream()),
          "mhcl_bwd_fused");
    link->y.reset();
    link->g_xout.reset();
    return {g_x, g_W, g_b, g_alpha, Tensor()};
  }
};

struct Post : Function<Post> {
  static Tensor forward(AutogradContext *ctx, Tensor x, Tensor y, Tensor H_res, Tensor H_post, LinkPtr link) {
    const Tensor yc = y.contiguous(), x_out = empty_stream(x, x.sizes(), 0);
    check(mhcl_post(&link->d, ptr(x), ptr(yc), ptr<float>(H_res), ptr<float>(H_post), ptr(x_out), stream()), "mhcl_post");
    ctx->save_for_backward({H_res, H_post});
    ctx->saved_data["link"] = keep(link);
    link->y = yc.detach();
    return x_out;
  }

  static variable_list backward(AutogradContext *ctx, variable_list grads) {
    const variable_list saved = ctx->get_saved_variables();
    const LinkPtr link = kept(ctx);
    const mhcl_desc &d = link->d;
    const Tensor g_xout = grads[0].contiguous().detach();
    link->g_xout = g_xout;
    const Tensor g_y = at::empty({d.T, d.C}, g_xout.options());
    // g_y = sum_i H_post[i] g_xout[i]
    check(mhcl_pre(&d, ptr(g_xout), ptr<float>(saved[1]), ptr(g_y), stream()), "mhcl_pre");
    // x and the coefficients get their gradients from the coefficient node (fused kernel), which
    // autograd runs once this node is done, also where no gradient reaches it through f
    return {Tensor(), g_y, Tensor(), Tensor(), Tensor()};
  }
};

// (gradients may come at any address; the kernels read 16 bytes at a time)
Tensor dense(const Tensor &t) {
  const Tensor c = t.contiguous();
  return (reinterpret_cast<uintptr_t>(c.data_ptr()) & 15u) == 0 ? c : c.clone();
}

// The ends of a stack: n copies of the input, the sum of the streams; each is the other's backward.
Tensor copies(const mhcl_desc &d, const Tensor &x0, int64_t phase) {
  const Tensor x = empty_stream(x0, {d.T, d.n, d.C}, phase);
  check(mhcl_streams_in(&d, ptr(x0), ptr(x), stream()), "mhcl_streams_in");
  return x;
}
Tensor sum(const mhcl_desc &d, const Tensor &x) {
  const Tensor out = at::empty({d.T, d.C}, x.options());
  check(mhcl_streams_out(&d, ptr(x), ptr(out), stream()), "mhcl_streams_out");
  return out;
}
struct StreamsIn : Function<StreamsIn> {
  static Tensor forward(AutogradContext *ctx, Tensor x0, LinkPtr link) {
    ctx->saved_data["link"] = keep(link);
    return copies(link->d, x0, 0);
  }
  static variable_list backward(AutogradContext *ctx, variable_list grads) {
    return {sum(kept(ctx)->d, dense(grads[0])), Tensor()};
  }
};
struct StreamsOut : Function<StreamsOut> {
  static Tensor forward(AutogradContext *ctx, Tensor x, LinkPtr link) {
    ctx->saved_data["link"] = keep(link);
    return sum(link->d, x);
  }
  static variable_list backward(AutogradContext *ctx, variable_list grads) {
    const LinkPtr link = kept(ctx);
    return {copies(link->d, dense(grads[0]), link->g_x_phase), Tensor()};
  }
};

// what layers of one shape have in common, ahead of the calls below; perm: the int8 table of a permutation subset
LinkPtr make_link(int64_t n, int64_t C, int64_t T, int io_dtype, int res_mode, int sk_iters, double eps,
                  const std::optional<Tensor> &perm, int64_t g_x_phase) {
  LinkPtr l = c10::make_intrusive<Link>();
  l->d = mhcl_desc{};
  l->d.n = static_cast<int32_t>(n);
  l->d.C = static_cast<int32_t>(C);
  l->d.T = T;
  l->d.io_dtype = io_dtype;
  l->d.res_mode = res_mode;
  l->d.sk_iters = sk_iters;
  l->d.eps = static_cast<float>(eps);
  if (perm) {
    // (as binding.Desc: the kernels index the table as [K][n])
    TORCH_CHECK_VALUE(perm->scalar_type() == at::kChar && perm->dim() == 2 && perm->size(1) == n && perm->is_contiguous(),
                      "perm must be a contiguous int8 tensor [K, n]");
    TORCH_CHECK_VALUE(T == 0 || perm->is_cuda(), "perm must be a GPU tensor");
    l->perm = *perm;
    l->d.n_perm = static_cast<int32_t>(perm->size(0));
    l->d.perm = static_cast<const int8_t *>(perm->data_ptr());
  }
  l->g_x_phase = g_x_phase;
  return l;
}

// whether x lies in memory as the kernels of a stack with input x0 read it
bool readable(const Tensor &x, const Tensor &x0, const LinkPtr &link) {
  const mhcl_desc &d = link->d;
  return x.layout() == at::kStrided && x.scalar_type() == x0.scalar_type() && x.device() == x0.device() && x.dim() == 3 &&
         x.size(0) == d.T && x.size(1) == d.n && x.size(2) == d.C && x.is_contiguous() && !x.is_neg() &&
         (reinterpret_cast<uintptr_t>(x.data_ptr()) & 15u) == 0;
}

std::tuple<Tensor, Tensor, Tensor> coeffs_pre(const Tensor &x, const Tensor &W, const Tensor &b, const Tensor &alpha,
                                              const LinkPtr &link) {
  const variable_list out = CoeffsPre::apply(x, W, b, alpha, link);
  return {out[0], out[1], out[2]};
}

}  // namespace

PYBIND11_MODULE(TORCH_EXTENSION_NAME, m) {
  // (Python exceptions go on to the caller; other threads run during the calls, as during torch's own: an allocation or a
  // launch may wait for the GPU, and the GPU for what another thread is to do)
  const auto wrap = [](auto f) { return torch::wrap_pybind_function_no_gil(f); };
  py::class_<Link, LinkPtr>(m, "Link");
  m.def("link", wrap(&make_link));
  m.def("coeffs_pre", wrap(&coeffs_pre));
  m.def("post", wrap([](const Tensor &x, const Tensor &y, const Tensor &H_res, const Tensor &H_post, const LinkPtr &link) {
          return Post::apply(x, y, H_res, H_post, link);
        }));
  m.def("streams_in", wrap([](const Tensor &x0, const LinkPtr &link) { return StreamsIn::apply(x0, link); }));
  m.def("readable", torch::wrap_pybind_function(&readable));
  m.def("streams_out", wrap([](const Tensor &x, const LinkPtr &link) { return StreamsOut::apply(x, link); }));
}
