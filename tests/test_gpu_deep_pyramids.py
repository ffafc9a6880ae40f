"""Levels above 6 on both sides of where the pyramids of tile sums lie in LDS (1184 tiles in the backward, 2400 in the forward) and beyond: output and
gradients against float64 with the filter in block-mean form.  float32: sums of up to 2^12 rows and of n rows in the gate's gradients, 1e-4;
bf16: 2e-2, the bars of the two paths."""
import pytest

pytestmark = pytest.mark.gpu


def blocks(x, l):
    """Sums of aligned blocks of 2^l rows, at every row."""
    import torch
    n = x.shape[2]
    w = 1 << l
    p = torch.nn.functional.pad(x, (0, 0, 0, -n % w))
    return p.unflatten(2, (-1, w)).sum(3, keepdim=True).expand(-1, -1, -1, w, -1).flatten(2, 3)[:, :, :n]


def reference(q, k, v, dout, omega, gw, gb, sw, L):
    import torch
    x = [t.double().requires_grad_(True) for t in (q, k, v, gw, gb, sw)]
    qd, kd, vd, gwd, gbd, swd = x
    f = torch.sigmoid(torch.einsum("hld,bhd->bhl", gwd, qd.mean(2)) + gbd) * swd

    def filt(t):
        out = f[..., 0][..., None, None] * t
        for l in range(1, L + 1):
            out = out + ((f[..., l] - f[..., l - 1]) / 2 ** l)[..., None, None] * blocks(t, l)
        return out

    pq, pk = (torch.relu(filt(t) @ omega.double()) / omega.shape[-1] ** 0.5 for t in (qd, kd))
    out = (pq @ (pk.transpose(2, 3) @ vd)) / (pq @ pk.sum(2)[..., None] + 1e-6)
    return [out.detach()] + list(torch.autograd.grad(out, x, dout.double()))


@pytest.mark.parametrize("dtype,d,m", [("f32", 16, 16), ("bf16", 64, 128)])
@pytest.mark.parametrize("n,L", [(65, 7), (75776, 12), (75777, 12), (153600, 9), (153601, 9)])
def test_deep_transform(dtype, d, m, n, L):
    import torch
    from paper_2507_08637_amd import binding
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator(device="cuda").manual_seed(n + d)
    wave = torch.sin(torch.arange(n, device="cuda") * (6.2832 / 2 ** (L - 1)))[:, None]   # something for the upper levels to carry

    def rows(a):
        return (torch.randn(1, 1, n, d, generator=g, device="cuda") + a * wave + 0.2).to(dt)

    q, k, v, dout = rows(0.7), rows(0.7), rows(1.0), rows(1.0)
    omega = torch.randn(d, m, generator=g, device="cuda").to(dt)
    gw = torch.randn(1, L + 1, d, generator=g, device="cuda") / d ** 0.5
    gb, sw = torch.randn(1, L + 1, generator=g, device="cuda"), 1 + 0.1 * torch.randn(L + 1, generator=g, device="cuda")
    one = torch.ones(1, device="cuda")
    out, saved = binding.wersa_forward(q, k, v, omega, one, gw, gb, sw, L)
    got = binding.wersa_backward(q, k, v, omega, one, gw, gb, sw, out, dout, saved, L)
    ref = reference(q, k, v, dout, omega, gw, gb, sw, L)
    names = ("out", "dq", "dk", "dv") + (("dgate_w", "dgate_b", "dscale_w") if dtype == "f32" and n > 65 else ())
    err = {x: float(((out if x == "out" else got[x]).double() - r).norm() / r.norm())
           for x, r in zip(("out", "dq", "dk", "dv", "dgate_w", "dgate_b", "dscale_w"), ref)}
    print((dtype, d, m, n, L), {x: f"{e:.1e}" for x, e in err.items()}, flush=True)
    assert all(err[x] < (1e-4 if dtype == "f32" else 2e-2) for x in names), err
