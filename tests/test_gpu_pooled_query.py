"""The pooled query (Section 3.1 step 4) bit for bit: four interleaved float32 sums over the partial sums of Q,
((s0 + s1) + (s2 + s3)) / n, whatever kernel adds them and with how many waves.  A last bit of it moves the filter and,
at rounding edges of the operands and of the ReLU's step, everything after.  One row per 64-row tile is not
zero, so that the partial sums of a transform deeper than one tile are exactly those rows."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _interleaved(parts, n):
    """parts (chunks, columns) float32."""
    acc = np.zeros((4, parts.shape[1]), dtype=np.float32)
    for c in range(parts.shape[0]):
        acc[c % 4] += parts[c]
    return ((acc[0] + acc[1]) + (acc[2] + acc[3])) / np.float32(n)


@pytest.mark.parametrize("flags", [0, 4], ids=["plain", "pooled_gate"])
@pytest.mark.parametrize("tiles", [1, 4, 31, 33, 100, 161, 400])
@pytest.mark.parametrize("dtype,d,m", [("bf16", 64, 128), ("bf16", 128, 128), ("f32", 16, 32), ("f32", 112, 32)])
def test_order_of_the_partial_sums(dtype, d, m, tiles, flags):
    import torch
    from paper_2507_08637_amd import binding
    B, H, L, n = 1, 3, 7, 64 * tiles - 5
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator(device="cuda").manual_seed(tiles * d)

    def normal(*s):
        return torch.randn(s, generator=g, device="cuda")

    q = torch.zeros(B, H, n, d, dtype=tdt, device="cuda")
    rows = (normal(B, H, tiles, d) * torch.exp(2 * normal(B, H, tiles, 1))).to(tdt)
    q[:, :, 7::64] = rows
    k, v = normal(B, H, n, d).to(tdt), normal(B, H, n, d).to(tdt)
    par = (normal(d, m).to(tdt), torch.ones(1, device="cuda"), normal(H, L + 1, d) / 8, normal(H, L + 1),
           torch.ones(L + 1, device="cuda"))
    _, saved = binding.wersa_forward(q, k, v, *par, L, flags=flags)
    qbar = binding.saved_views(binding.make_desc(q, L, m, flags=flags), saved)["qbar"].cpu().numpy()
    for h in range(H):
        want = _interleaved(rows[0, h].float().cpu().numpy(), n)
        assert np.array_equal(qbar[h], want), (h, np.abs(qbar[h] - want).max())
