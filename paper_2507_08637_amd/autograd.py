"""torch.autograd bindings of the WERSA hot path (argument marshalling only: every step runs in
the HIP kernels behind the C ABI).

    out = wersa_attention(q, k, v, omega_rf, sigma, gate_w, gate_b, scale_w, L)
    y = wersa_attention_block(x, wq, wk, wv, wo, H, omega_rf, sigma, gate_w, gate_b, scale_w, L)

q, k, v: (B, H, n, d) with a shared layout (any strides, last dimension contiguous); gradients
flow to q, k, v, sigma, gate_w, gate_b, scale_w (omega_rf is a fixed random matrix) and, for the
block, to x and the four weight matrices (float32 gradients cast to the weights' dtype).
"""
import ctypes
import warnings

import torch

from . import binding


_node = None   # (False: it does not load)


def _load_node():
    """The extension that holds the attention core's node of the autograd graph (csrc/wersa_torch.cpp), on the library that the
    binding has loaded.  It is bound to one version of torch where the library is not: without it the node in Python makes the same
    calls, and a warning says that its host path is the slower one."""
    global _node
    if _node is None:
        lib = binding.load_library()
        try:
            from . import _wersa_torch as node
        except ImportError as e:
            warnings.warn("the autograd extension _wersa_torch.so is missing or does not load, training steps take up to 100 us longer on "
                          f"the host: build it with `python -m paper_2507_08637_amd.build` ({e})", RuntimeWarning, stacklevel=3)
            _node = False
            return _node
        node.bind(*(ctypes.cast(f, ctypes.c_void_p).value for f in (lib.wersa_forward, lib.wersa_backward, lib.wersa_workspace_bytes,
                                                                    lib.wersa_saved_bytes, lib.wersa_selected_path)))
        _node = node
    return _node


class _WersaAttention(torch.autograd.Function):
    """The same node in Python, for torch.jit.trace (the tracer records its call, and of the one in C++ only the allocation of the output) and where
    the extension does not load."""

    @staticmethod
    def forward(ctx, q, k, v, omega_rf, sigma, gate_w, gate_b, scale_w, L, eps, bw_floor):
        out, saved = binding.wersa_forward(q, k, v, omega_rf, sigma, gate_w, gate_b, scale_w, L, eps=eps,
                                           bw_floor=bw_floor)
        ctx.save_for_backward(q, k, v, omega_rf, sigma, gate_w, gate_b, scale_w, out, saved)
        ctx.cfg = (L, eps, bw_floor, q.stride())
        return out

    @staticmethod
    def backward(ctx, dout):
        q, k, v, omega_rf, sigma, gate_w, gate_b, scale_w, out, saved = ctx.saved_tensors
        L, eps, bw_floor, strides = ctx.cfg
        # (saved-tensor hooks may have made them dense; `saved` is laid out for the path that the forward's strides select)
        q, k, v, out, dout = (x if x.stride() == strides else torch.empty_strided(x.shape, strides, dtype=x.dtype, device=x.device).copy_(x)
                              for x in (q, k, v, out, dout))
        g = binding.wersa_backward(q, k, v, omega_rf, sigma, gate_w, gate_b, scale_w, out, dout, saved, L,
                                   eps=eps, bw_floor=bw_floor)
        return (g["dq"], g["dk"], g["dv"], None, g["dsigma"], g["dgate_w"], g["dgate_b"], g["dscale_w"],
                None, None, None)


def wersa_attention(q, k, v, omega_rf, sigma, gate_w, gate_b, scale_w, L, eps=1e-6, bw_floor=1e-6):
    node = _load_node() if _node is None else _node
    if not node or torch.jit.is_tracing():
        return _WersaAttention.apply(q, k, v, omega_rf, sigma, gate_w, gate_b, scale_w, L, eps, bw_floor)
    desc, saved_bytes, workspace = binding.checked_desc(q, k, v, omega_rf, sigma, gate_w, gate_b, scale_w, L, eps, bw_floor, 0)
    return node.attention(q, k, v, omega_rf, sigma, gate_w, gate_b, scale_w, bytes(desc), saved_bytes, workspace)


class _WersaBlock(torch.autograd.Function):
    @staticmethod
    def forward(ctx, x, wq, wk, wv, wo, H, omega_rf, sigma, gate_w, gate_b, scale_w, L, eps, bw_floor):
        y, saved = binding.wersa_block_forward(x, wq, wk, wv, wo, H, omega_rf, sigma, gate_w, gate_b, scale_w, L,
                                               eps=eps, bw_floor=bw_floor)
        ctx.save_for_backward(x, wq, wk, wv, wo, omega_rf, sigma, gate_w, gate_b, scale_w, saved)
        ctx.cfg = (H, L, eps, bw_floor)
        return y

    @staticmethod
    def backward(ctx, dy):
        x, wq, wk, wv, wo, omega_rf, sigma, gate_w, gate_b, scale_w, saved = ctx.saved_tensors
        H, L, eps, bw_floor = ctx.cfg
        g = binding.wersa_block_backward(x, wq, wk, wv, wo, H, omega_rf, sigma, gate_w, gate_b, scale_w,
                                         dy.contiguous(), saved, L, eps=eps, bw_floor=bw_floor)
        cast = lambda t: t.to(wq.dtype)
        return (g["dx"], cast(g["dwq"]), cast(g["dwk"]), cast(g["dwv"]), cast(g["dwo"]), None, None, g["dsigma"],
                g["dgate_w"], g["dgate_b"], g["dscale_w"], None, None, None)


def wersa_attention_block(x, wq, wk, wv, wo, H, omega_rf, sigma, gate_w, gate_b, scale_w, L, eps=1e-6,
                          bw_floor=1e-6):
    return _WersaBlock.apply(x, wq, wk, wv, wo, H, omega_rf, sigma, gate_w, gate_b, scale_w, L, eps, bw_floor)
