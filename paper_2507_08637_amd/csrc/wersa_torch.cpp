// The attention core as a node of torch's autograd graph, in C++: what a training step pays for on the host beyond the launches.  The engine runs
// a backward on a thread of its own, and interpreter state, reference counts and runtime structures that both threads touch move between their
// caches at every change.  2 x 4 slices of 1000 tokens, d 64, m 256, bf16, forward and backward: 235 to 246 us where the engine's thread runs far from
// the caller's and 128 to 136 where near with a node written in Python, 128 to 138 and 98 with this one; its kernels take 97.
//
// The library is reached through the addresses of its entry points (bind): this module has no link to it, and loads whichever the
// binding loaded.  The forward's arguments are checked by the caller, what the backward unpacks is checked here; the library checks the
// rest, and its status is raised as the binding's error.
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
decltype(&wersa_workspace_bytes) workspace_bytes_fn = nullptr;
decltype(&wersa_saved_bytes) saved_bytes_fn = nullptr;
decltype(&wersa_selected_path) selected_path_fn = nullptr;

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

// Raises AssertionError, as the binding's checks do, unless `holds`.
void require(bool holds, const char *text) {
  if (holds) return;
  pybind11::gil_scoped_acquire gil;
  PyErr_SetString(PyExc_AssertionError, text);
  python_error err;
  err.persist();
  throw err;
}

// (host tensors have no stream: entry points that only note their arguments are given such)
void *stream(const Tensor &t) { return t.is_cuda() ? (void *)c10::hip::getCurrentHIPStream().stream() : nullptr; }
Tensor scratch(int64_t bytes, const Tensor &like) {
  return at::empty({bytes < 256 ? 256 : bytes}, like.options().dtype(at::kByte));
}
const float *floats(const Tensor &t) { return static_cast<const float *>(t.const_data_ptr()); }
float *floats_out(const Tensor &t) { return static_cast<float *>(t.mutable_data_ptr()); }

bool same_layout(const Tensor &a, const Tensor &b) { return a.sizes() == b.sizes() && a.strides() == b.strides() && a.dtype() == b.dtype(); }
bool holds_floats(const Tensor &t, int64_t count) { return t.dtype() == at::kFloat && t.is_contiguous() && t.numel() >= count; }

struct Attention : torch::autograd::Function<Attention> {
  static Tensor forward(AutogradContext *ctx, const Tensor &q, const Tensor &k, const Tensor &v, const Tensor &omega, const Tensor &sigma,
                        const Tensor &gate_w, const Tensor &gate_b, const Tensor &scale_w, const std::string &desc, int64_t saved_bytes,
                        int64_t workspace) {
    const wersa_desc d = desc_of(desc);
    const Tensor out = at::empty_strided(q.sizes(), q.strides(), q.options());
    const Tensor saved = at::empty({saved_bytes / 4}, q.options().dtype(at::kFloat));
    const Tensor ws = scratch(workspace, q);
    check(forward_fn(&d, q.const_data_ptr(), k.const_data_ptr(), v.const_data_ptr(), omega.const_data_ptr(), floats(sigma), floats(gate_w),
                     floats(gate_b), floats(scale_w), out.mutable_data_ptr(), saved.mutable_data_ptr(), ws.mutable_data_ptr(), ws.nbytes(),
                     stream(q)));
    ctx->save_for_backward({q, k, v, omega, sigma, gate_w, gate_b, scale_w, out, saved});
    ctx->saved_data["desc"] = desc;
    return out;
  }

  // Saved-tensor hooks may give the tensors back in another layout than the forward had them in (save_on_cpu makes them dense, or contiguous):
  // the call, its workspace and its outputs are described by the tensors that are there now.
  static variable_list backward(AutogradContext *ctx, const variable_list &grads) {
    const variable_list t = ctx->get_saved_variables();
    Tensor q = t[0], k = t[1], v = t[2], out = t[8], dout = grads[0];
    const Tensor &omega = t[3], &sigma = t[4], &gate_w = t[5], &gate_b = t[6], &scale_w = t[7], &saved = t[9];
    const wersa_desc then = desc_of(ctx->saved_data["desc"].toStringRef());
    wersa_desc d = then;
    require(q.dim() == 4 && q.sizes() == at::IntArrayRef({d.B, d.H, d.n, d.d}) && q.stride(3) == 1 &&
                q.dtype() == (d.dtype == WERSA_F32 ? at::kFloat : at::kBFloat16),
            "expect q as it was saved: (B, H, n, d) with contiguous last dim");
    d.stride_b = q.stride(0), d.stride_h = q.stride(1), d.stride_n = q.stride(2);
    require(same_layout(q, k) && same_layout(q, v) && same_layout(q, out), "q, k, v, out and gradients must share shape, strides and dtype");
    const int path = selected_path_fn(&d);
    if (path >= 0 && path != selected_path_fn(&then)) {   // `saved` is laid out for the other path (strides of 8 elements or not): back to its strides
      d = then;
      for (Tensor *x : {&q, &k, &v, &out}) *x = at::empty_strided(x->sizes(), {d.stride_b, d.stride_h, d.stride_n, 1}, x->options()).copy_(*x);
    }
    auto like_q = [&]() { return at::empty_strided(q.sizes(), q.strides(), q.options()); };
    if (dout.strides() != q.strides()) dout = like_q().copy_(dout);
    require(same_layout(q, dout), "q, k, v, out and gradients must share shape, strides and dtype");
    const int64_t matrices = d.flags & WERSA_FLAG_SEPARATE_OMEGA ? 2 : 1;
    require(omega.is_contiguous() && omega.dtype() == q.dtype() && omega.numel() == matrices * d.d * d.m &&
                holds_floats(sigma, 1) && holds_floats(gate_w, (int64_t)d.H * (d.L + 1) * d.d) && holds_floats(gate_b, (int64_t)d.H * (d.L + 1)) &&
                holds_floats(scale_w, d.L + 1),
            "expect omega and the parameters as they were saved");
    require(holds_floats(saved, (int64_t)saved_bytes_fn(&d) / 4), "the saved buffer holds less than wersa_saved_bytes asks for");
    for (const Tensor &x : t) require(x.device() == dout.device(), "saved tensors on another device");
    const Tensor dq = like_q(), dk = like_q(), dv = like_q(), dgw = at::empty_like(gate_w), dgb = at::empty_like(gate_b),
                 dsw = at::empty_like(scale_w), dsg = at::empty({1}, sigma.options());
    const Tensor ws = scratch((int64_t)workspace_bytes_fn(&d, 1), q);
    check(backward_fn(&d, q.const_data_ptr(), k.const_data_ptr(), v.const_data_ptr(), omega.const_data_ptr(), floats(sigma), floats(gate_w),
                      floats(gate_b), floats(scale_w), out.const_data_ptr(), dout.const_data_ptr(), saved.const_data_ptr(), dq.mutable_data_ptr(),
                      dk.mutable_data_ptr(), dv.mutable_data_ptr(), floats_out(dgw), floats_out(dgb), floats_out(dsw), floats_out(dsg),
                      ws.mutable_data_ptr(), ws.nbytes(), stream(q)));
    return {dq, dk, dv, Tensor(), dsg, dgw, dgb, dsw, Tensor(), Tensor(), Tensor()};
  }
};

Tensor attention(const Tensor &q, const Tensor &k, const Tensor &v, const Tensor &omega, const Tensor &sigma, const Tensor &gate_w,
                 const Tensor &gate_b, const Tensor &scale_w, const pybind11::bytes &desc, int64_t saved_bytes, int64_t workspace) {
  const std::string d = desc;
  pybind11::gil_scoped_release nogil;
  return Attention::apply(q, k, v, omega, sigma, gate_w, gate_b, scale_w, d, saved_bytes, workspace);
}

}  // namespace

PYBIND11_MODULE(_wersa_torch, m) {
  m.def("bind", [](uintptr_t forward, uintptr_t backward, uintptr_t workspace_bytes, uintptr_t saved_bytes, uintptr_t selected_path) {
    forward_fn = reinterpret_cast<decltype(forward_fn)>(forward);
    backward_fn = reinterpret_cast<decltype(backward_fn)>(backward);
    workspace_bytes_fn = reinterpret_cast<decltype(workspace_bytes_fn)>(workspace_bytes);
    saved_bytes_fn = reinterpret_cast<decltype(saved_bytes_fn)>(saved_bytes);
    selected_path_fn = reinterpret_cast<decltype(selected_path_fn)>(selected_path);
  });
  m.def("attention", &attention);
}
