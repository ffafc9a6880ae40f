"""MFMA path with several row groups per workgroup of the rows and gradient kernels (asserted) and, at head dimension 128, eight waves per
contraction workgroup: partial last blocks, transforms above one block, and the options with separate random matrices for queries
and keys, against the library's own float32 arithmetic (WERSA_FLAG_GENERIC_PATH) on the same inputs.  Bounds as in the tests of partial
last blocks: 6e-3 for O and dV, 2e-2 for dQ and dK.  Rows past the sequence must come out untouched."""
import pytest

pytestmark = pytest.mark.gpu

CASES = [  # B, H, n, d, m, L, flags
    (12, 4, 4100, 64, 256, 4, 0), (12, 4, 4100, 64, 256, 9, 0), (12, 4, 4100, 64, 384, 4, 0), (12, 4, 4100, 64, 384, 9, 8),
    (16, 4, 1100, 128, 256, 6, 0), (16, 4, 1100, 128, 256, 8, 0), (16, 4, 1121, 128, 384, 6, 0), (16, 4, 1121, 128, 512, 8, 0),
    (16, 4, 1088, 128, 512, 6, 2), (16, 4, 1088, 128, 512, 6, 14), (16, 4, 1100, 128, 512, 6, 14), (16, 4, 1100, 128, 384, 5, 2),
    (12, 4, 4096, 64, 256, 5, 14), (12, 4, 4100, 64, 256, 5, 2),
]


@pytest.mark.parametrize("B,H,n,d,m,L,flags", CASES)
def test_against_float32_arithmetic(B, H, n, d, m, L, flags):
    import torch
    from paper_2507_08637_amd import binding
    groups, pad = -(-n // (512 if d == 64 else 256)), 70
    assert groups > max(256 // (B * H), 1)
    g = torch.Generator(device="cuda").manual_seed(n + d + m + L + flags)

    def normal(*s):
        return torch.randn(s, generator=g, device="cuda")

    def place(t=None):   # (B, H, n, d) inside a buffer with `pad` rows behind each sequence, all of them 7
        buf = torch.full((B, H, n + pad, d), 7.0, dtype=torch.bfloat16, device="cuda")
        if t is not None:
            buf[:, :, :n].copy_(t)
        return buf, buf[:, :, :n]

    # rows on a slow wave, values and their gradients with profiles over the columns, so that dQ is no small difference of large terms
    t, j = torch.arange(n, device="cuda")[:, None], 2 * torch.pi * torch.arange(d, device="cuda") / d
    wave = torch.sin(2 * torch.pi * t / 256)
    q, k = (place(normal(B, H, n, d) + 0.7 * wave + 0.2)[1] for _ in range(2))
    v, dout = (place(0.3 * normal(B, H, n, d) + wave * torch.cos(j + a) + torch.cos((3 - a) * j))[1] for a in (0, 1))
    gw, gb, sw = normal(H, L + 1, d) / d ** 0.5, 0.5 * normal(H, L + 1), 1 + 0.1 * normal(L + 1)
    omega = normal(*((2, d, m) if flags & 2 else (d, m))).to(torch.bfloat16)   # two: nothing in common
    par = (omega, torch.ones(1, device="cuda"), gw, gb, sw)
    assert binding.load_library().wersa_selected_path(binding.make_desc(q, L, m, flags=flags)) == 1
    res = {}
    for path in (0, binding.FLAG_GENERIC_PATH):
        fl = dict(flags=flags | path, eps=1e-3)
        obuf, out = place()
        _, saved = binding.wersa_forward(q, k, v, *par, L, out=out, **fl)
        bufs = {name: place() for name in ("dq", "dk", "dv")}
        grads = dict({name: b[1] for name, b in bufs.items()}, dgate_w=torch.empty_like(gw), dgate_b=torch.empty_like(gb),
                     dscale_w=torch.empty_like(sw), dsigma=torch.empty(1, device="cuda"))
        binding.wersa_backward(q, k, v, *par, out, dout, saved, L, grads=grads, **fl)
        for name, (buf, _) in dict(bufs, out=(obuf, out)).items():
            assert bool((buf[:, :, n:] == 7.0).all()), (name, path)
        res[path] = dict(grads, out=out)
    errs = {}
    for name in ("out", "dq", "dk", "dv"):
        a, r = res[0][name].double(), res[binding.FLAG_GENERIC_PATH][name].double()
        errs[name] = float((a - r).norm() / r.norm())
    print((B, H, n, d, m, L, flags), {x: f"{e:.1e}" for x, e in errs.items()}, flush=True)
    assert errs["out"] < 6e-3 and errs["dv"] < 6e-3 and errs["dq"] < 2e-2 and errs["dk"] < 2e-2, errs
