"""The attention block's matrix products, each against a float32 product of the same stored operands:
Q', K', V', Y, dA, dX (bf16: one rounding of a float32 sum, 2^-9 relative at most, 2e-3 with the sums'
own error) and the weight gradients (float32: sums of up to 24576 products of bf16 values with unit
roundoff 2^-24 per addition in the worst order of magnitude sqrt(24576) 2^-24 = 1e-5)."""
import pytest

pytestmark = pytest.mark.gpu

SHAPES = [
    # B, H, n, d: 128-wide workgroup tiles; one row panel group and a partial one; the last split shorter
    (1, 4, 256, 64),
    (5, 4, 256, 64),
    (3, 8, 768, 64),
    (1, 16, 1792, 64),
    # 256-wide tiles for the three projections only, for every product, 13 and 9 row panels (groups of four)
    (1, 16, 5632, 128),
    (3, 16, 4352, 128),
    (1, 8, 24576, 64),
    # 256-wide tiles of eight steps, 97 per XCD on 32 workgroups: four of them in one workgroup and three in the others
    (1, 4, 65792, 64),
    # products with a weight's transpose on transposed copies (from 32768 tokens on): hidden no power of two
    (1, 12, 32768, 64),
    # weight gradients: 31 splits of nine steps and one of a single step, two tiles per workgroup
    (1, 16, 8960, 64),
]


@pytest.mark.parametrize("offset", [0, 1], ids=["aligned", "misaligned"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "B{}H{}n{}d{}".format(*s))
def test_products(shape, offset):
    import torch
    from paper_2507_08637_amd import binding
    B, H, n, d = shape
    hidden, L, m = H * d, 3, 128
    g = torch.Generator(device="cuda").manual_seed(B * n + offset)

    def bf(*s, scale=1.0):   # a contiguous tensor `offset` elements into its allocation
        buf = torch.empty(offset + int(torch.Size(s).numel()), dtype=torch.bfloat16, device="cuda")
        buf[offset:] = (scale * torch.randn(s, generator=g, device="cuda")).to(torch.bfloat16).flatten()
        return buf[offset:].view(s)

    x, dy = bf(B, n, hidden), bf(B, n, hidden)
    w = [bf(hidden, hidden, scale=hidden ** -0.5) for _ in range(4)]
    omega = torch.randn(d, m, generator=g, device="cuda").to(torch.bfloat16)
    sigma = torch.ones(1, device="cuda")
    gw = torch.randn(H, L + 1, d, generator=g, device="cuda") / 8
    gb = torch.randn(H, L + 1, generator=g, device="cuda")
    sw = torch.ones(L + 1, device="cuda")
    args = (H, omega, sigma, gw, gb, sw)
    y, saved = binding.wersa_block_forward(x, *w, *args, L)
    desc = binding.make_block_desc(x, H, L, m)
    ws = torch.empty(binding.load_library().wersa_block_workspace_bytes(desc, 1), dtype=torch.uint8, device="cuda")
    gr = binding.wersa_block_backward(x, *w, *args, dy, saved, L, workspace=ws)
    sv, wv = binding.block_saved_views(desc, saved), binding.block_workspace_views(desc, ws)

    def flat(t):
        return t.float().reshape(-1, hidden)

    def rel(a, ref):
        return float((flat(a).double() - ref.double()).norm() / ref.double().norm())

    wf = [t.float() for t in w]
    want = dict(Qp=flat(x) @ wf[0], Kp=flat(x) @ wf[1], Vp=flat(x) @ wf[2], Y=flat(sv["A"]) @ wf[3],
                dA=flat(dy) @ wf[3].t(),
                dX=flat(wv["dQp"]) @ wf[0].t() + flat(wv["dKp"]) @ wf[1].t() + flat(wv["dVp"]) @ wf[2].t())
    got = dict(Qp=sv["Qp"], Kp=sv["Kp"], Vp=sv["Vp"], Y=y, dA=wv["dA"], dX=gr["dx"])
    errs = {k: rel(got[k], want[k]) for k in want}
    grads = dict(dwo=(sv["A"], dy), dwq=(x, wv["dQp"]), dwk=(x, wv["dKp"]), dwv=(x, wv["dVp"]))
    gerr = {k: rel(gr[k], flat(a).t() @ flat(b)) for k, (a, b) in grads.items()}
    # the pooled query comes out of the W^Q product's epilogue (or of a pass over Q' where the core pools by itself)
    core = sv["core"]
    core_desc = binding.WersaDesc(B, H, n, d, L, m, 1, 1e-6, 1e-6, n * hidden, d, hidden, 0)
    at = binding.load_library().wersa_saved_offset(core_desc, 2)
    qbar = core[at:at + B * H * d].view(B, hidden)
    qerr = float((qbar - want["Qp"].view(B, n, hidden).mean(1)).norm() / want["Qp"].std() * n ** 0.5 / qbar.numel() ** 0.5)
    print(shape, offset, errs, gerr, f"qbar {qerr:.1e}", flush=True)
    assert all(v < 2e-3 for v in errs.values()), errs
    assert all(v < 1e-5 for v in gerr.values()), gerr
    assert qerr < 4e-3   # of the mean's own standard deviation: one bf16 rounding per row at most
