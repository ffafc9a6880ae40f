"""The ReLU's decisions that the backward's contraction and dV kernels leave as bits for the gradient kernels (MFMA path): every bit is
seen.  Rows and random features of +-1 with an odd number of non-zero columns and a transform of no levels make every
pre-activation an odd multiple of the filter's one coefficient: no decision is at the edge of a rounding, and a row of dQ or dK
misses or has too much by one of about m / 2 terms where a bit is wrong, sqrt(2 / m) >= 5.5e-2 of its norm (m <= 640).  Against
float64: rounding of dPhi's 2^-9 per term, of O and of the row itself, below 2e-2 of a row's norm.

FEW slices: one 64-row block per contraction workgroup and one row group per workgroup of the gradient kernels.  MANY slices: several of
both (asserted), so that running offsets, requests for the next group and words read anew in every pass are seen, and eight waves
per contraction workgroup at head dimension 128 with whole 256s of features."""
import pytest

pytestmark = pytest.mark.gpu

# tiles of 32 and 64 rows, up to 17 groups of 512 or 256 rows; 128 and 256 features per pass, one to five passes
FEW = ([(6 if n <= 4000 else 3, n, 64, m) for n, m in ((32, 256), (64, 128), (97, 384), (513, 256), (1000, 512), (1025, 640), (8200, 256), (8200, 128))]
       + [(6 if n <= 4000 else 3, n, 128, m) for n, m in ((32, 256), (65, 128), (257, 384), (1000, 512), (4100, 256))])
MANY = ([(96, n, 64, m) for n, m in ((1088, 128), (1100, 256), (1100, 384), (1088, 512))]
        + [(64, n, 128, m) for n, m in ((1088, 256), (1100, 256), (1100, 384), (1121, 512))])


def reference(q, k, v, dout, omega, sigma, gw, gb, sw, eps, layernorm):
    import torch
    x = [t.double().requires_grad_(True) for t in (q, k, v)]
    qd, kd, vd = x
    f = torch.sigmoid(torch.einsum("hd,bhd->bh", gw[:, 0].double(), qd.mean(2)) + gb[:, 0].double()) * sw.double()
    om = omega.double() / sigma.double() / omega.shape[-1] ** 0.5
    pq, pk = (torch.relu((f[..., None, None] * t) @ om) for t in (qd, kd))
    s, z = pk.transpose(2, 3) @ vd, pk.sum(2)
    out = pq @ s
    if layernorm:
        out = (out - out.mean(-1, keepdim=True)) / (out.var(-1, unbiased=False, keepdim=True) + eps).sqrt()
    else:
        out = out / (pq @ z[..., None] + eps)
    return torch.autograd.grad(out, x, dout.double())


def plan(slices, n, d, m):
    """Blocks per contraction workgroup and row groups of a gradient kernel's workgroup with the most: the library's split."""
    blocks = -(-n // 64)
    features = 256 if d == 64 and m % 256 == 0 else 128
    want = min(max(512 // (slices * (m // features)), 1), blocks)
    groups = -(-n // (512 if d == 64 else 256))
    return -(-blocks // want), -(-groups // min(max(256 // slices, 1), groups))


@pytest.mark.parametrize("slices,n,d,m,flags", [c + (0,) for c in FEW + MANY] + [c + (8,) for c in MANY])
def test_every_decision(slices, n, d, m, flags):
    import torch
    from paper_2507_08637_amd import binding
    B, H, L = slices // 3, 3, 0
    if slices > 6:
        B, H = slices // 4, 4
        assert min(plan(slices, n, d, m)) >= 2
    g = torch.Generator(device="cuda").manual_seed(n + d + m)

    def normal(*s):
        return torch.randn(s, generator=g, device="cuda")

    q, k, omega = ((1 - 2 * (normal(*s) < 0).float()).to(torch.bfloat16) for s in ((B, H, n, d), (B, H, n, d), (d, m)))
    omega[0] = 0   # 63 or 127 columns count
    v, dout = (normal(B, H, n, d).to(torch.bfloat16) for _ in range(2))
    sigma, gw, gb, sw = torch.ones(1, device="cuda"), normal(H, 1, d) / d ** 0.5, normal(H, 1), torch.ones(1, device="cuda")
    assert binding.load_library().wersa_selected_path(binding.make_desc(q, L, m)) == 1
    out, saved = binding.wersa_forward(q, k, v, omega, sigma, gw, gb, sw, L, flags=flags)
    got = binding.wersa_backward(q, k, v, omega, sigma, gw, gb, sw, out, dout, saved, L, flags=flags)
    ref = reference(q, k, v, dout, omega, sigma, gw, gb, sw, 1e-6, flags == 8)
    worst = {}
    for name, r in zip(("dq", "dk", "dv"), ref):
        e = (got[name].double() - r).norm(dim=-1) / r.norm(dim=-1).clamp_min(0.1 * float(r.norm(dim=-1).mean()))
        worst[name] = float(e.max())
    print((slices, n, d, m, flags), {x: f"{e:.1e}" for x, e in worst.items()}, flush=True)
    assert max(worst.values()) < 2e-2, worst


@pytest.mark.parametrize("n,m", [(131072, 256), (131072, 128), (65544, 256)])
def test_queries_decide_as_the_forward(n, m):
    """Head dimension 64: dQ uses the decisions that the forward's rows kernel takes, bit for bit: the filtered queries that leave the bits are summed in
    that kernel's order.  The key side's decisions come from a rows kernel, so a problem with Q = K that is the same on both sides must give
    the same decisions on both: one value per slice for all of V and dO and an eps far above the normaliser make the two gradients of a
    feature equal (d z_r / eps) up to rounding.  A feature's decision is read from a column of its own (0 in Q, 1 in its
    column of Omega).  The signal's columns are constant over 64 rows and their band is weighted with 1e-3 against the others' 1.4, so
    that the filter's sums cancel and a sum in another order gives other bits, and some other decisions: one is worth up to 1 of `size` in its row,
    rounding a few times 2^-9."""
    import torch
    from paper_2507_08637_amd import binding
    H, d, L, tags = 8, 64, 6, 56
    g = torch.Generator(device="cuda").manual_seed(n + m + L)

    def normal(*s):
        return torch.randn(s, generator=g, device="cuda")

    q = torch.zeros(1, H, n, d, device="cuda")
    q[..., tags:] = normal(1, H, -(-n // 2 ** L), 8).repeat_interleave(2 ** L, 2)[:, :, :n]
    q = q.to(torch.bfloat16)
    omega = torch.zeros(d, m, device="cuda")
    omega[tags:, :tags] = normal(8, tags)
    omega[:tags, :tags] = torch.eye(tags, device="cuda")
    omega = omega.to(torch.bfloat16)
    ones = torch.ones_like(q)
    scale = torch.full((L + 1,), 2.7913, device="cuda")
    scale[L] = 2.1e-3
    par = (torch.ones(1, device="cuda"), torch.zeros(H, L + 1, d, device="cuda"), torch.zeros(H, L + 1, device="cuda"), scale)
    opt = dict(eps=1e6)
    assert binding.load_library().wersa_selected_path(binding.make_desc(q, L, m)) == 1
    out, saved = binding.wersa_forward(q, q, ones, omega, *par, L, **opt)
    got = binding.wersa_backward(q, q, ones, omega, *par, out, ones, saved, L, **opt)
    z = binding.saved_views(binding.make_desc(q, L, m, eps=1e6), saved)["z"].double()[:, :tags]
    size = 0.5 * float(scale[0]) * d * z / 1e6 / m ** 0.5   # of a feature's decision, in its column of dQ
    assert float(size.min()) > 0
    differ = (got["dq"].double() - got["dk"].double())[0, ..., :tags].abs().amax(1) / size
    mixed = (got["dk"][0, ..., :tags].double().abs().amax(1) / size > 0.5).sum()   # features whose rows of a block do not all agree
    print((n, m), f"worst {float(differ.max()):.1e}, mixed {int(mixed)} of {size.numel()}", flush=True)
    assert int(mixed) > 10   # (otherwise nothing is seen)
    assert float(differ.max()) < 0.1
