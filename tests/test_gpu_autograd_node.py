"""The attention core's node of the autograd graph: what the engine, its hooks and transforms make of it.  Gradients are compared with the
binding's own backward on the same tensors: the same kernels, so the same bits."""
import pytest

pytestmark = pytest.mark.gpu

NAMES = ("q", "k", "v", "sigma", "gate_w", "gate_b", "scale_w")


def problem(layout="bhnd", n=200, dtype="bf16"):
    import torch
    g = torch.Generator(device="cuda").manual_seed(n)
    B, H, d, L, m = 2, 3, 64, 3, 128
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32

    def normal(*s):
        return torch.randn(s, generator=g, device="cuda")

    def rows():
        x = (normal(B, H, n, d) + 0.3).to(dt)
        return x if layout == "bhnd" else x.permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3)

    t = dict(q=rows(), k=rows(), v=rows(), omega=normal(d, m).to(dt), sigma=torch.ones(1, device="cuda"), gate_w=normal(H, L + 1, d) / 8,
             gate_b=normal(H, L + 1), scale_w=1 + 0.1 * normal(L + 1))
    return t, rows(), L


def direct(t, dout, L):
    from paper_2507_08637_amd import binding
    import torch
    a = [t[x].detach() for x in ("q", "k", "v", "omega", "sigma", "gate_w", "gate_b", "scale_w")]
    out, saved = binding.wersa_forward(*a, L)
    d = torch.empty_strided(out.shape, out.stride(), dtype=out.dtype, device=out.device).copy_(dout)
    g = binding.wersa_backward(*a, out, d, saved, L)
    return out, [g["dq"], g["dk"], g["dv"], g["dsigma"], g["dgate_w"], g["dgate_b"], g["dscale_w"]]


def node(t, L):
    from paper_2507_08637_amd.autograd import wersa_attention
    return wersa_attention(*(t[x] for x in ("q", "k", "v", "omega", "sigma", "gate_w", "gate_b", "scale_w")), L)


def same(a, b):
    import torch
    assert len(a) == len(b) and all(x.dtype == y.dtype and torch.equal(x, y) for x, y in zip(a, b))


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("layout", ["bhnd", "bnhd"])
@pytest.mark.parametrize("dout", ["like", "other", "expanded"])
def test_gradients_are_the_bindings(dtype, layout, dout):
    import torch
    t, g, L = problem(layout, dtype=dtype)
    if dout == "other":
        g = g.contiguous() if layout == "bnhd" else g.transpose(1, 2).contiguous().transpose(1, 2)
    elif dout == "expanded":
        g = g[..., :1].expand(g.shape)
    for x in NAMES:
        t[x].requires_grad_(True)
    out = node(t, L)
    ref, grads = direct(t, g, L)
    assert out.stride() == t["q"].stride() and torch.equal(out, ref)
    for _ in range(2):
        same(torch.autograd.grad(out, [t[x] for x in NAMES], g, retain_graph=True), grads)


def test_some_inputs_side_stream_and_another_thread():
    import threading
    import torch
    t, g, L = problem()
    _, grads = direct(t, g, L)
    with torch.no_grad():
        assert not node(t, L).requires_grad
    assert not node(t, L).requires_grad
    t["k"].requires_grad_(True)
    t["gate_b"].requires_grad_(True)
    got = {}

    def step():
        s = torch.cuda.Stream()
        s.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(s):
            (node(t, L).float() * g.float()).sum().backward()
        s.synchronize()
        got.update(k=t["k"].grad, b=t["gate_b"].grad)

    torch.cuda.synchronize()
    th = threading.Thread(target=step)
    th.start()
    th.join()
    same([got["k"], got["b"]], [grads[1], grads[5]])
    assert t["q"].grad is None


def test_saved_tensor_hooks_and_versions():
    import torch
    t, g, L = problem()
    for x in NAMES:
        t[x].requires_grad_(True)
    packed = []

    def pack(x):
        packed.append(x)
        return x.detach().cpu()

    with torch.autograd.graph.saved_tensors_hooks(pack, lambda x: x.cuda()):
        out = node(t, L)
    assert len(packed) >= 8
    same(torch.autograd.grad(out, [t[x] for x in NAMES], g), direct(t, g, L)[1])
    out = node(t, L)
    with torch.no_grad():
        t["v"].add_(1)
    with pytest.raises(RuntimeError, match="modified by an inplace operation"):
        torch.autograd.grad(out, [t["q"]], g)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("hook", ["on_cpu", "pinned", "contiguous"])
@pytest.mark.parametrize("layout", ["bnhd", "fused", "odd"])
def test_saved_tensors_that_come_back_in_another_layout(layout, hook, dtype):
    """fused: slices of one projection's output; odd: rows d + 1 elements apart, which in bf16 is another path than dense rows take."""
    import torch
    t, g, L = problem("bnhd", dtype=dtype)
    B, H, n, d = g.shape
    if layout != "bnhd":
        wide = torch.empty(B, n, 3 * H * d if layout == "fused" else 3 * H * (d + 1), dtype=g.dtype, device="cuda").view(B, n, 3, H, -1)
        for i, x in enumerate("qkv"):
            wide[:, :, i, :, :d] = t[x].permute(0, 2, 1, 3)
            t[x] = wide[:, :, i, :, :d].permute(0, 2, 1, 3)
    for x in NAMES:
        t[x] = t[x].detach().requires_grad_(True)
    ref, grads = direct(t, g, L)
    if hook == "contiguous":
        hooks = torch.autograd.graph.saved_tensors_hooks(lambda x: x.detach().clone(memory_format=torch.contiguous_format), lambda x: x)
    else:
        hooks = torch.autograd.graph.save_on_cpu(pin_memory=hook == "pinned")
    with hooks:
        out = node(t, L)
    assert torch.equal(out, ref)
    for _ in range(2):
        same(torch.autograd.grad(out, [t[x] for x in NAMES], g, retain_graph=True), grads)


def test_traced_module():
    import torch
    t, g, L = problem("bnhd")
    names = ("q", "k", "v", "omega", "sigma", "gate_w", "gate_b", "scale_w")
    traced = torch.jit.trace(lambda *a: node(dict(zip(names, a)), L), [t[x] for x in names])
    u = {x: (t[x] * 0.75).requires_grad_(x in NAMES) for x in names}
    ref, grads = direct(u, g, L)
    for _ in range(3):
        out = traced(*(u[x] for x in names))
        assert torch.equal(out, ref)
        same(torch.autograd.grad(out, [u[x] for x in NAMES], g), grads)


def test_what_is_refused():
    import torch
    from paper_2507_08637_amd import binding
    from paper_2507_08637_amd.autograd import wersa_attention
    t, g, L = problem()
    rest = [t[x] for x in ("k", "v", "omega", "sigma", "gate_w", "gate_b", "scale_w")]
    with pytest.raises(RuntimeError):   # transforms
        torch.func.vmap(lambda q: wersa_attention(q, *rest, L))(t["q"][None].repeat(2, 1, 1, 1, 1))
    with pytest.raises(RuntimeError):
        torch.func.grad(lambda q: wersa_attention(q, *rest, L).float().sum())(t["q"])
    import torch.autograd.forward_ad as fwd
    with fwd.dual_level():
        with pytest.raises((RuntimeError, NotImplementedError)):
            wersa_attention(fwd.make_dual(t["q"], g), *rest, L)
    with pytest.raises(AssertionError):
        wersa_attention(t["q"][:, :, 1:], *rest, L)
    with pytest.raises(TypeError):
        wersa_attention(*(x.double() if i < 3 else x for i, x in enumerate([t["q"]] + rest)), L)
    off = torch.empty(t["q"].numel() + 1, dtype=torch.bfloat16, device="cuda")[1:].view(t["q"].shape)   # 2 bytes past 16
    with pytest.raises(binding.WersaError) as e:
        wersa_attention(off, *rest, L)
    assert e.value.status == 1
    with pytest.raises(binding.WersaError):
        wersa_attention(t["q"], *rest, 99)
