"""Sums over a row's columns in the LayerNorm output stage (MFMA path): small terms beside large ones are kept."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [64, 65])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("pair", [(0, 1), (8, 9), (5, 37), (31, 62)])
def test_small_columns_beside_two_large_ones(n, d, pair):
    """Every row of N is n v with v = (1, -1) in two columns and +-s in the others, s^2 just below 2^-23, exactly: one query and one key row
    over and over, features that are all 1, powers of two elsewhere.  Added one by one to the two squares (2), the others are less than half a
    unit in its last place and are lost, 30 of 64 columns and 62 of 128 where a lane adds its half of the row: 9e-7 and 1.8e-6 of
    1 / sqrt(var + eps).  Added pairwise, at most six roundings meet the large terms, 2^-24 of the sum each, half of that after the
    square root; the root and the division add 2^-22 at most."""
    import torch
    from paper_2507_08637_amd import binding
    m, L, eps = 256, 0, 1e-6
    s = 0.99609375 * 2.0 ** -11.5   # (rounded to bf16 below)
    v = torch.full((d,), s, dtype=torch.float64).to(torch.bfloat16).double()
    v[::2] *= -1
    a, b = pair
    v[a], v[b] = 1.0, -1.0
    rest = [j for j in range(d) if j not in pair]
    v[rest] = v[rest].abs() * torch.tensor([1.0, -1.0], dtype=torch.float64).repeat(len(rest) // 2)
    assert float(v.sum()) == 0.0 and 0.9 * 2.0 ** -23 < float(v[rest[0]]) ** 2 < 2.0 ** -23
    q = torch.zeros(1, 1, n, d, device="cuda", dtype=torch.bfloat16)
    q[..., 0] = 1
    vals = v.to(torch.bfloat16).cuda().expand(1, 1, n, d).contiguous()
    vals[:, :, 64:] = 0   # (S stays a power of two times v)
    omega = torch.zeros(d, m, device="cuda", dtype=torch.bfloat16)
    omega[0] = 1
    one = torch.ones(1, device="cuda")
    par = (one, torch.zeros(1, L + 1, d, device="cuda"), torch.zeros(1, L + 1, device="cuda"), 2 * one)
    flags = binding.FLAG_LAYERNORM
    assert binding.load_library().wersa_selected_path(binding.make_desc(q, L, m, flags=flags)) == 1
    out, saved = binding.wersa_forward(q, q, vals, omega, *par, L, eps=eps, flags=flags)
    rstd = binding.saved_views(binding.make_desc(q, L, m, eps, flags=flags), saved)["D"].double().cpu()[0]
    ref = 1.0 / ((64 * v).square().mean() + torch.tensor(eps).double()).sqrt()
    err = float((rstd / ref - 1).abs().max())
    print((n, d, pair), f"{err:.1e}", flush=True)
    assert err < 6 * 2.0 ** -25 + 2.0 ** -22
    assert float((out[0, 0].double().cpu() - 64 * v * ref).abs().max()) < 2.0 ** -8 * float(64 * ref)
