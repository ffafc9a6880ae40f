"""The attention core's node of the autograd graph on the CPU, its library calls replaced by entry points that note what they are given:
what a backward is told about tensors that come back from saved-tensor hooks in another layout."""
import ctypes
import warnings
from contextlib import contextmanager

import pytest
import torch

from paper_2507_08637_amd import autograd, binding

B, H, N, D, L, M = 2, 4, 100, 64, 3, 128


@contextmanager
def recorded(forward_status=0, backward_status=0):
    """Calls of wersa_forward and wersa_backward: (descriptor, addresses and sizes)."""
    lib, calls = binding.load_library(), []

    def entry(like, status):
        proto = ctypes.CFUNCTYPE(ctypes.c_int, ctypes.POINTER(binding.WersaDesc), *like.argtypes[1:])

        def call(desc, *args):
            calls.append((binding.WersaDesc.from_buffer_copy(desc.contents), args))
            return status
        return proto(call)

    node = autograd._load_node()
    fakes = entry(lib.wersa_forward, forward_status), entry(lib.wersa_backward, backward_status)
    address = lambda f: ctypes.cast(f, ctypes.c_void_p).value
    rest = [address(f) for f in (lib.wersa_workspace_bytes, lib.wersa_saved_bytes, lib.wersa_selected_path)]
    node.bind(*(address(f) for f in fakes), *rest)
    try:
        yield calls
    finally:
        node.bind(address(lib.wersa_forward), address(lib.wersa_backward), *rest)


def tensors(layout, dtype=torch.bfloat16):
    if layout == "fused":      # slices of one projection's output
        q, k, v = torch.randn(B, N, 3 * H * D).to(dtype).view(B, N, 3, H, D).permute(2, 0, 3, 1, 4)
    elif layout == "odd":      # rows that are no multiple of eight elements apart: not for the MFMA path
        q, k, v = (torch.randn(B, H, N, D + 1).to(dtype)[..., :D] for _ in range(3))
    else:
        q, k, v = (torch.randn(B, N, H, D).to(dtype).permute(0, 2, 1, 3) for _ in range(3))
        if layout == "bhnd":
            q, k, v = (x.contiguous() for x in (q, k, v))
    params = [torch.randn(D, M).to(dtype), torch.ones(1), torch.randn(H, L + 1, D), torch.randn(H, L + 1), torch.ones(L + 1)]
    return [x.detach().requires_grad_(True) for x in (q, k, v)], params


def contiguous(x):
    return x.detach().clone(memory_format=torch.contiguous_format)


HOOKS = {"none": None, "contiguous": contiguous, "dense": lambda x: x.detach().clone(memory_format=torch.preserve_format)}


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("hook", HOOKS)
@pytest.mark.parametrize("layout", ["bhnd", "bnhd", "fused", "odd"])
def test_backward_describes_the_tensors_that_are_there(layout, hook, dtype):
    qkv, params = tensors(layout, dtype)
    unpacked = {}

    def unpack(x):
        unpacked[x.data_ptr()] = x
        return x

    with recorded() as calls:
        if hook == "none":
            out = autograd.wersa_attention(*qkv, *params, L)
            for x in (*qkv, out):
                unpacked[x.data_ptr()] = x
        else:
            with torch.autograd.graph.saved_tensors_hooks(HOOKS[hook], unpack):
                out = autograd.wersa_attention(*qkv, *params, L)
        assert out.stride() == qkv[0].stride()
        for dout in (torch.ones_like(out), torch.ones(B, H, N, 1, dtype=dtype).expand(out.shape)):
            grads = torch.autograd.grad(out, qkv, dout, retain_graph=True)
            desc, args = calls[-1]
            strides = (desc.stride_b, desc.stride_h, desc.stride_n)
            lib = binding.load_library()
            assert binding.wersa_path_name(desc) == binding.wersa_path_name(calls[0][0])   # the path that laid `saved` out
            assert args[-2] >= lib.wersa_workspace_bytes(ctypes.byref(desc), 1)
            assert [g.stride()[:3] for g in grads] == [strides] * 3 and [g.data_ptr() for g in grads] == list(args[11:14])
            others = [desc.B, desc.H, desc.n, desc.d, desc.m, desc.L, desc.dtype, desc.flags]
            assert others == [B, H, N, D, M, L, int(dtype == torch.bfloat16), 0]
            if layout == "odd" and hook != "none" and dtype == torch.bfloat16:   # copied back to where the forward's path had them
                assert strides == qkv[0].stride()[:3] and not set(args[:3]) & set(unpacked)
            else:
                assert [unpacked[a].stride()[:3] for a in (*args[:3], args[8])] == [strides] * 4


@pytest.mark.parametrize("index,change", [
    (1, lambda x: x.transpose(1, 2).contiguous().transpose(1, 2)), (2, lambda x: x.float()), (8, lambda x: x[:, :, 1:]),
    (0, lambda x: x[..., ::2].repeat_interleave(2, -1).transpose(2, 3).contiguous().transpose(2, 3)), (3, lambda x: x.float()), (3, lambda x: x[:, 1:]),
    (4, lambda x: x.double()), (5, lambda x: x.transpose(1, 2).contiguous().transpose(1, 2)), (6, lambda x: x[:1]), (7, lambda x: x.half()),
    (9, lambda x: x[:-1])])
def test_tensors_that_came_back_otherwise_are_refused(index, change):
    """q, k, v, omega, sigma, gate_w, gate_b, scale_w, out, saved: one of them in another layout, size or type than the call can take."""
    qkv, params = tensors("bhnd")
    seen = []

    def pack(x):
        seen.append(x)
        return len(seen) - 1, x.detach()

    with recorded() as calls:
        with torch.autograd.graph.saved_tensors_hooks(pack, lambda p: change(p[1]) if p[0] == index else p[1]):
            out = autograd.wersa_attention(*qkv, *params, L)
        assert len(seen) == 10
        with pytest.raises(AssertionError):
            torch.autograd.grad(out, qkv, torch.ones_like(out))
    assert len(calls) == 1


@pytest.mark.parametrize("index", range(10))
def test_a_tensor_that_came_back_on_another_device_is_refused(index):
    qkv, params = tensors("bhnd")
    seen = []

    def pack(x):
        seen.append(x)
        return len(seen) - 1, x.detach()

    with recorded() as calls:
        with torch.autograd.graph.saved_tensors_hooks(pack, lambda p: p[1].to("meta") if p[0] == index else p[1]):
            out = autograd.wersa_attention(*qkv, *params, L)
        with pytest.raises(AssertionError, match="device"):
            torch.autograd.grad(out, qkv, torch.ones_like(out))
    assert len(calls) == 1


def test_status_of_either_call_is_raised():
    qkv, params = tensors("bhnd")
    with recorded(forward_status=3):
        with pytest.raises(binding.WersaError) as e:
            autograd.wersa_attention(*qkv, *params, L)
        assert e.value.status == 3
    with recorded(backward_status=1):
        out = autograd.wersa_attention(*qkv, *params, L)
        with pytest.raises(binding.WersaError) as e:
            torch.autograd.grad(out, qkv, torch.ones_like(out))
        assert e.value.status == 1


def test_traced_module_makes_the_call(monkeypatch):
    """A traced module runs the attention on its own inputs; the library's calls are replaced by ones that compute something on the CPU."""
    def forward(q, k, v, omega, sigma, gate_w, gate_b, scale_w, L, **kw):
        return (q + 2 * k + 3 * v) * scale_w[L], torch.zeros(1)

    def backward(q, k, v, omega, sigma, gate_w, gate_b, scale_w, out, dout, saved, L, **kw):
        s = scale_w[L]
        return dict(dq=dout * s, dk=2 * dout * s, dv=3 * dout * s, dsigma=torch.zeros(1), dgate_w=torch.zeros_like(gate_w),
                    dgate_b=torch.zeros_like(gate_b), dscale_w=torch.zeros_like(scale_w))

    monkeypatch.setattr(binding, "wersa_forward", forward)
    monkeypatch.setattr(binding, "wersa_backward", backward)
    qkv, params = tensors("bnhd", torch.float32)
    with recorded():
        traced = torch.jit.trace(lambda q, k, v, *p: autograd.wersa_attention(q, k, v, *p, L), (*qkv, *params), check_trace=False)
    qkv, params = tensors("bnhd", torch.float32)
    params[4] = torch.full((L + 1,), 0.5)
    out = traced(*qkv, *params)
    assert torch.equal(out, forward(*qkv, *params, L)[0])
    grads = torch.autograd.grad(out, qkv, torch.ones_like(out))
    assert [float(g.mean()) for g in grads] == [0.5, 1.0, 1.5]


@pytest.mark.parametrize("hook", ["contiguous", "dense"])
@pytest.mark.parametrize("layout", ["bnhd", "fused", "odd"])
def test_node_in_python_goes_back_to_the_strides_of_the_forward(monkeypatch, layout, hook):
    """The node that a trace records: tensors that come back in another layout may select another path than the one that laid saved out."""
    seen = []

    def forward(q, *a, **kw):
        return torch.empty_strided(q.shape, q.stride(), dtype=q.dtype).zero_(), torch.zeros(1)

    def backward(q, k, v, omega, sigma, gate_w, gate_b, scale_w, out, dout, saved, L, **kw):
        seen.extend((q, k, v, out, dout))
        return dict(dq=q, dk=k, dv=v, dsigma=sigma, dgate_w=gate_w, dgate_b=gate_b, dscale_w=scale_w)

    monkeypatch.setattr(binding, "wersa_forward", forward)
    monkeypatch.setattr(binding, "wersa_backward", backward)
    qkv, params = tensors(layout)
    with torch.autograd.graph.saved_tensors_hooks(HOOKS[hook], lambda x: x):
        out = autograd._WersaAttention.apply(*qkv, *params, L, 1e-6, 1e-6)
    grads = torch.autograd.grad(out, qkv, torch.ones(B, H, N, 1, dtype=out.dtype).expand(out.shape))
    assert [x.stride() for x in seen] == [qkv[0].stride()] * 5 and all(torch.equal(g, x) for g, x in zip(grads, qkv))


def test_without_the_extension_the_node_in_python_makes_the_calls(monkeypatch):
    """libwersa.so alone suffices; one warning."""
    import sys
    import paper_2507_08637_amd as package
    made = []

    def forward(q, k, v, *a, **kw):
        made.append("forward")
        return q + k + v, torch.zeros(1)

    def backward(q, k, v, omega, sigma, gate_w, gate_b, scale_w, out, dout, saved, L, **kw):
        made.append("backward")
        return dict(dq=dout, dk=2 * dout, dv=3 * dout, dsigma=sigma, dgate_w=gate_w, dgate_b=gate_b, dscale_w=scale_w)

    monkeypatch.delattr(package, "_wersa_torch", raising=False)
    monkeypatch.setitem(sys.modules, "paper_2507_08637_amd._wersa_torch", None)
    monkeypatch.setattr(autograd, "_node", None)
    monkeypatch.setattr(binding, "wersa_forward", forward)
    monkeypatch.setattr(binding, "wersa_backward", backward)
    qkv, params = tensors("bhnd")
    with pytest.warns(RuntimeWarning, match="_wersa_torch.so"):
        out = autograd.wersa_attention(*qkv, *params, L)
    grads = torch.autograd.grad(out, qkv, torch.ones_like(out))
    assert [float(g.float().mean()) for g in grads] == [1, 2, 3]
    with warnings.catch_warnings():
        warnings.simplefilter("error")
        autograd.wersa_attention(*qkv, *params, L)
    assert made == ["forward", "backward", "forward"]
