"""The gate of the forward where the first kernel that filters forms it (head dimension 64 on the MFMA path; few packing workgroups on the split
path) and on both sides of where it is a launch of its own: pooled query, sigmoids and filter as `saved` keeps them, against float64.  Sums
of n terms of size one in float32 chunks: a few times 2^-24 sqrt(n) / n absolute in the mean, and a logit is a sum of d of them: 1e-5."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,B,H,n,d,L,m", [
    ("bf16", 1, 1, 40, 64, 0, 128),          # one partial sum
    ("bf16", 2, 3, 1025, 64, 6, 256),        # two; a band more than twice the waves
    ("bf16", 1, 1, 131072, 64, 5, 128),      # 128 of them, the most
    ("bf16", 1, 1, 131073, 64, 5, 128),      # 129: a launch of its own
    ("f32", 1, 1, 16, 16, 1, 16),
    ("f32", 2, 3, 2000, 48, 4, 64),          # 32 partial sums, columns padded to 64
    ("f32", 1, 2, 4100, 128, 6, 32),         # 65: sixteen chains of four and five
    ("f32", 2, 5, 4300, 64, 3, 32),          # 2040 packing workgroups
    ("f32", 2, 5, 4400, 64, 3, 32),          # 2070: a launch of its own
    ("bf16", 3, 2, 300, 16, 2, 96),
])
def test_gate_against_float64(dtype, B, H, n, d, L, m):
    import torch
    from paper_2507_08637_amd import binding
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator(device="cuda").manual_seed(n + d + L)

    def normal(*s):
        return torch.randn(s, generator=g, device="cuda")

    q, k, v = ((normal(B, H, n, d) + 0.3).to(dt) for _ in range(3))
    omega, gw, gb = normal(d, m).to(dt), normal(H, L + 1, d) / d ** 0.5, 0.5 * normal(H, L + 1)
    sw, sigma = 1 + 0.1 * normal(L + 1), torch.ones(1, device="cuda")
    _, saved = binding.wersa_forward(q, k, v, omega, sigma, gw, gb, sw, L)
    got = binding.saved_views(binding.make_desc(q, L, m), saved)
    qbar = q.double().mean(2)
    s = torch.sigmoid(torch.einsum("hld,bhd->bhl", gw.double(), qbar) + gb.double())
    for name, ref in (("qbar", qbar), ("s", s), ("F", s * sw.double())):
        err = float((got[name].double() - ref.reshape(got[name].shape)).abs().max())
        print((dtype, B, H, n, d, L), name, f"{err:.1e}", flush=True)
        assert err < 1e-5, name
