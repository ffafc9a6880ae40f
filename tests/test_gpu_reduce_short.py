"""Sum of the contraction's partial results by threads that take all partials of their columns (MFMA path, 128 workgroups of 1024 outputs and
more): numbers of partials around the eight that are in flight together, the feature counts that fill a part of z's last workgroup, and the case just
below the line.  S, z and what the forward makes of their bf16 copies against float64; operands rounded to 2^-9 and 2^-11, so that a sum of
like terms is off by 2^-9 at most and O by as much again: 6e-3.  V has a mean, so that S is such a sum and a missing partial is a share of it."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("slices,d,m,partials", [(16, 64, 128, p) for p in (1, 2, 7, 8, 9, 15, 17, 32)] + [(15, 64, 128, 9)]
                         + [(8, 128, 128, p) for p in (1, 3, 8, 13)] + [(8, 128, 384, 5), (3, 64, 1152, 6), (33, 64, 640, 3)])
def test_sum_of_partials(slices, d, m, partials):
    import torch
    from paper_2507_08637_amd import binding
    n, L = 64 * partials, 0
    g = torch.Generator(device="cuda").manual_seed(partials + m)

    def normal(*s):
        return torch.randn(s, generator=g, device="cuda")

    q, k, v = (x.to(torch.bfloat16) for x in (normal(1, slices, n, d), normal(1, slices, n, d), 1 + 0.5 * normal(1, slices, n, d)))
    omega = normal(d, m).to(torch.bfloat16)
    one = torch.ones(1, device="cuda")
    gw, gb = torch.zeros(slices, 1, d, device="cuda"), torch.zeros(slices, 1, device="cuda")
    assert binding.load_library().wersa_selected_path(binding.make_desc(q, L, m)) == 1
    out, saved = binding.wersa_forward(q, k, v, omega, one, gw, gb, 2 * one, L)   # filter 1
    got = binding.saved_views(binding.make_desc(q, L, m), saved)
    pq, pk = (torch.relu(x[0].double() @ omega.double()) / m ** 0.5 for x in (q, k))
    S, z = pk.transpose(1, 2) @ v[0].double(), pk.sum(1)
    O = (pq @ S) / (pq @ z[..., None])
    for name, a, b in (("S", got["S"], S), ("z", got["z"], z), ("O", out[0], O)):
        err = float((a.double() - b).norm() / b.norm())
        print((slices, d, m, partials), name, f"{err:.1e}", flush=True)
        assert err < 6e-3, name
