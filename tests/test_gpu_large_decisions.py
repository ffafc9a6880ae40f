"""MFMA path: one buffer for the ReLU's decisions of both sides (tensors from 512 MiB on), the query side first."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,m,n,H,flags", [(64, 128, 524288, 8, 0), (64, 256, 599200, 7, 8), (128, 128, 131104, 16, 0)])
def test_one_buffer_for_both_sides(d, m, n, H, flags):
    """Against the float32-arithmetic path.  Bounds: those of the bf16 tests; a side that read the other's decisions would be off by 1 / sqrt(2) or so."""
    import torch
    from paper_2507_08637_amd import binding
    L = 4
    g = torch.Generator(device="cuda").manual_seed(m)

    def normal(*s):
        return torch.randn(s, generator=g, device="cuda")

    # rows on a slow wave, values and their gradients with profiles over the columns: O, and with it dQ, is not the small
    # difference of large terms that independent values would give
    t, j = torch.arange(n, device="cuda")[:, None], 2 * torch.pi * torch.arange(d, device="cuda") / d
    wave = torch.sin(2 * torch.pi * t / 256)
    q, k = ((normal(1, H, n, d) + 0.7 * wave + 0.2).to(torch.bfloat16) for _ in range(2))
    v, dout = ((0.3 * normal(1, H, n, d) + wave * torch.cos(j + a) + torch.cos((3 - a) * j)).to(torch.bfloat16) for a in (0, 1))
    par = (normal(d, m).to(torch.bfloat16), torch.ones(1, device="cuda"), normal(H, L + 1, d) / d ** 0.5, normal(H, L + 1), 1 + 0.1 * normal(L + 1))
    assert H * n * d * 2 >= 512 << 20
    got = []
    for f in (flags, flags | binding.FLAG_GENERIC_PATH):
        out, saved = binding.wersa_forward(q, k, v, *par, L, eps=1e-3, flags=f)
        got.append(dict(binding.wersa_backward(q, k, v, *par, out, dout, saved, L, eps=1e-3, flags=f), out=out))
    errs = {x: float((got[0][x].float() - got[1][x].float()).norm() / got[1][x].float().norm()) for x in ("out", "dq", "dk", "dv")}
    print((d, m, n, H, flags), {x: f"{e:.1e}" for x, e in errs.items()}, flush=True)
    assert errs["out"] < 1e-2 and errs["dv"] < 1e-2 and errs["dq"] < 3e-2 and errs["dk"] < 3e-2, errs
