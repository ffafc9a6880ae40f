"""The ReLU's decisions that the split path's contraction (and at head dimension 128 the kernel of dV) leaves as bits for its gradient kernels:
every bit is seen, as in test_gpu_relu_bits.py: +-1 in an odd number of columns, so that no pre-activation is near zero, and a row of dQ or dK
misses or has too much by one of about m / 2 terms where a bit is wrong, sqrt(2 / m) >= 5.5e-2 of its norm.  Against float64: float32 1e-4
(sums of some hundred terms and their differences), bf16 results and O rounded to 2^-9, below 2e-2 of a row's norm; behind the LayerNorm
output stage the rounding of O enters dN = rstd (dO - mean dO - O mean(dO O)) twice with 2^-9 |dO| rstd, and a row counts as no smaller than a
tenth of the mean row: 2 2^-9 / 0.1 + 1e-2 = 5e-2, a third of a wrong bit (m <= 96 there).  Sizes: workgroups of two and of four waves with one token
tile per wave, and with two (d 16 and 32: from 1024 workgroups on); partial last tiles of 32 and blocks of 64 rows; 3 to 17 feature tiles and a partial one."""
import pytest

from tests.test_gpu_relu_bits import reference

pytestmark = pytest.mark.gpu

SHAPES = ([(6, n, d, m) for d in (16, 32, 64, 128) for n, m in ((31, 96), (65, 80), (1000, 544))]
          + [(256, n, d, 96) for d in (16, 32) for n in (250, 470, 512)] + [(256, 300, 64, 96), (64, 300, 128, 96)])


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("slices,n,d,m,flags", [c + (0,) for c in SHAPES] + [c + (8,) for c in SHAPES if c[1] in (65, 470)])
def test_every_decision(slices, n, d, m, flags, dtype):
    import torch
    from paper_2507_08637_amd import binding
    B, H, L = slices // 2, 2, 0
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator(device="cuda").manual_seed(n + d + m)

    def normal(*s):
        return torch.randn(s, generator=g, device="cuda")

    q, k, omega = ((1 - 2 * (normal(*s) < 0).float()).to(dt) for s in ((B, H, n, d), (B, H, n, d), (d, m)))
    omega[0] = 0   # d - 1 columns count
    v, dout = (normal(B, H, n, d).to(dt) for _ in range(2))
    sigma, gw, gb, sw = torch.ones(1, device="cuda"), normal(H, 1, d) / d ** 0.5, normal(H, 1), torch.ones(1, device="cuda")
    f = flags | binding.FLAG_GENERIC_PATH
    out, saved = binding.wersa_forward(q, k, v, omega, sigma, gw, gb, sw, L, flags=f)
    got = binding.wersa_backward(q, k, v, omega, sigma, gw, gb, sw, out, dout, saved, L, flags=f)
    ref = reference(q, k, v, dout, omega, sigma, gw, gb, sw, 1e-6, flags == 8)
    worst = {}
    for name, r in zip(("dq", "dk", "dv"), ref):
        e = (got[name].double() - r).norm(dim=-1) / r.norm(dim=-1).clamp_min(0.1 * float(r.norm(dim=-1).mean()))
        worst[name] = float(e.max())
    print((slices, n, d, m, flags, dtype), {x: f"{e:.1e}" for x, e in worst.items()}, flush=True)
    assert max(worst.values()) < (1e-4 if dtype == "f32" else 5e-2 if flags == 8 else 2e-2), worst
