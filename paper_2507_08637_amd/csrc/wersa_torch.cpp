// The attention core as a node of torch's autograd graph, in C++: what a training step pays for on the host beyond the launches.  The engine runs
// a backward on a thread of its own, and interpreter state, reference counts and runtime structures that both threads touch move between their
// caches at every change.  2 x 4 slices of 1000 tokens, d 64, m 256, bf16, forward and backward: 235 to 246 us where the engine's thread runs far from
// the caller's and 128 to 136 where near with a node written in Python, 128 to 138 and 98 with this one; its kernels take 97.
//
// The library is reached through the addresses of its entry points (bind): this module has no link to it, and loads whichever the
// binding loaded.  Arguments are checked by the caller; the library checks the rest, and its status is raised as the binding's error.
#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/custom_function.h>
#include <torch/csrc/utils/pybind.h>

#include <cstring>

#include "../../include/wersa.h"

namespace {

using at::Tensor;
using torch::autograd::AutogradContext;
using torch::autograd::variable_list;

decltype(&wersa_forward) forward_fn = nullptr;
decltype(&wersa_backward) backward_fn = nullptr;

wersa_desc desc_of(const std::string &bytes) {
  wersa_desc d;
  TORCH_CHECK(bytes.size() == sizeof(d), "descriptor of another size");
  std::memcpy(&d, bytes.data(), sizeof(d));
  return d;
}

// Raises WersaError(status) in whichever thread this is.
void check(wersa_status status) {
  if (status == WERSA_OK) return;
  pybind11::gil_scoped_acquire gil;
  try {
    pybind11::module_::import("paper_2507_08637_amd.binding").attr("_check")((int)status);
  } catch (pybind11::error_already_set &e) {
    e.restore();
    python_error err;
    err.persist();
    throw err;
  }
}

void *stream() { return (void *)c10::hip::getCurrentHIPStream().stream(); }
Tensor scratch(int64_t bytes, const Tensor &like) {
  return at::empty({bytes < 256 ? 256 : bytes}, like.options().dtype(at::kByte));
}
const float *floats(const Tensor &t) { return static_cast<const float *>(t.const_data_ptr()); }
float *floats_out(const Tensor &t) { return static_cast<float *>(t.mutable_data_ptr()); }

struct Attention : torch::autograd::Function<Attention> {
  static Tensor forward(AutogradContext *ctx, const Tensor &q, const Tensor &k, const Tensor &v, const Tensor &omega, const Tensor &sigma,
                        const Tensor &gate_w, const Tensor &gate_b, const Tensor &scale_w, const std::string &desc, int64_t saved_bytes,
                        int64_t workspace, int64_t backward_workspace) {
    const wersa_desc d = desc_of(desc);
    const Tensor out = at::empty_strided(q.sizes(), q.strides(), q.options());
    const Tensor saved = at::empty({saved_bytes / 4}, q.options().dtype(at::kFloat));
    const Tensor ws = scratch(workspace, q);
    check(forward_fn(&d, q.const_data_ptr(), k.const_data_ptr(), v.const_data_ptr(), omega.const_data_ptr(), floats(sigma), floats(gate_w),
                     floats(gate_b), floats(scale_w), out.mutable_data_ptr(), saved.mutable_data_ptr(), ws.mutable_data_ptr(), ws.nbytes(),
                     stream()));
    ctx->save_for_backward({q, k, v, omega, sigma, gate_w, gate_b, scale_w, out, saved});
    ctx->saved_data["desc"] = desc;
    ctx->saved_data["workspace"] = backward_workspace;
    return out;
  }

  static variable_list backward(AutogradContext *ctx, const variable_list &grads) {
    const variable_list t = ctx->get_saved_variables();
    const Tensor &q = t[0], &k = t[1], &v = t[2], &omega = t[3], &sigma = t[4], &gate_w = t[5], &gate_b = t[6], &scale_w = t[7], &out = t[8],
                 &saved = t[9];
    const wersa_desc d = desc_of(ctx->saved_data["desc"].toStringRef());
    auto like_q = [&]() { return at::empty_strided(q.sizes(), q.strides(), q.options()); };
    Tensor dout = grads[0];
    if (dout.strides() != q.strides()) dout = like_q().copy_(dout);
    TORCH_CHECK(dout.sizes() == q.sizes() && dout.dtype() == q.dtype() && out.strides() == q.strides(),
                "q, k, v, out and gradients must share shape, strides and dtype");
    const Tensor dq = like_q(), dk = like_q(), dv = like_q(), dgw = at::empty_like(gate_w), dgb = at::empty_like(gate_b),
                 dsw = at::empty_like(scale_w), dsg = at::empty({1}, sigma.options());
    const Tensor ws = scratch(ctx->saved_data["workspace"].toInt(), q);
    check(backward_fn(&d, q.const_data_ptr(), k.const_data_ptr(), v.const_data_ptr(), omega.const_data_ptr(), floats(sigma), floats(gate_w),
                      floats(gate_b), floats(scale_w), out.const_data_ptr(), dout.const_data_ptr(), saved.const_data_ptr(), dq.mutable_data_ptr(),
                      dk.mutable_data_ptr(), dv.mutable_data_ptr(), floats_out(dgw), floats_out(dgb), floats_out(dsw), floats_out(dsg),
                      ws.mutable_data_ptr(), ws.nbytes(), stream()));
    return {dq, dk, dv, Tensor(), dsg, dgw, dgb, dsw, Tensor(), Tensor(), Tensor(), Tensor()};
  }
};

Tensor attention(const Tensor &q, const Tensor &k, const Tensor &v, const Tensor &omega, const Tensor &sigma, const Tensor &gate_w,
                 const Tensor &gate_b, const Tensor &scale_w, const pybind11::bytes &desc, int64_t saved_bytes, int64_t workspace,
                 int64_t backward_workspace) {
  const std::string d = desc;
  pybind11::gil_scoped_release nogil;
  return Attention::apply(q, k, v, omega, sigma, gate_w, gate_b, scale_w, d, saved_bytes, workspace, backward_workspace);
}

}  // namespace

PYBIND11_MODULE(_wersa_torch, m) {
  m.def("bind", [](uintptr_t forward, uintptr_t backward) {
    forward_fn = reinterpret_cast<decltype(forward_fn)>(forward);
    backward_fn = reinterpret_cast<decltype(backward_fn)>(backward);
  });
  m.def("attention", &attention);
}
