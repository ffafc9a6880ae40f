"""The pooled query (Section 3.1 step 4) of the MFMA path bit for bit: four interleaved float32 sums over the partial sums of Q,
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
@pytest.mark.parametrize("d", [64, 128])
def test_order_of_the_partial_sums(d, tiles, flags):
    import torch
    from paper_2507_08637_amd import binding
    B, H, L, n, m = 1, 3, 7, 64 * tiles - 5, 128
    tdt = torch.bfloat16
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


@pytest.mark.parametrize("shape", [(1, 4, 256, 64), (1, 8, 2048, 64), (1, 8, 16384, 128)], ids=lambda s: "B{}H{}n{}d{}".format(*s))
def test_order_of_the_block_columns(shape):
    """The attention block's W^Q product leaves the column sums of 128 rows of Q': per half of every 8-row group one
    chain over the rows, then the two halves, with the small and with the large workgroup tile alike.  W^Q = 1, so that
    Q' = X exactly."""
    import torch
    from paper_2507_08637_amd import binding
    B, H, n, d = shape
    hidden, L, m = H * d, 5, 128
    g = torch.Generator(device="cuda").manual_seed(n)

    def normal(*s):
        return torch.randn(s, generator=g, device="cuda")

    x = (normal(B, n, hidden) * torch.exp(normal(B, n, 1))).to(torch.bfloat16)
    w = [torch.eye(hidden, device="cuda").to(torch.bfloat16)] + [(normal(hidden, hidden) / hidden ** 0.5).to(torch.bfloat16) for _ in range(3)]
    par = (normal(d, m).to(torch.bfloat16), torch.ones(1, device="cuda"), normal(H, L + 1, d) / 8, normal(H, L + 1),
           torch.ones(L + 1, device="cuda"))
    _, saved = binding.wersa_block_forward(x, *w, H, *par, L)
    core = binding.block_saved_views(binding.make_block_desc(x, H, L, m), saved)["core"]
    at = binding.load_library().wersa_saved_offset(binding.WersaDesc(B, H, n, d, L, m, 1, 1e-6, 1e-6, n * hidden, d, hidden, 0), 2)
    qbar = core[at:at + hidden].cpu().numpy()
    # rows of one 128-row block as [8-row group][half][4]
    rows = x[0].float().cpu().numpy().reshape(n // 128, 16, 2, 4, hidden).transpose(0, 2, 1, 3, 4).reshape(n // 128, 2, 64, hidden)
    half = np.zeros((n // 128, 2, hidden), dtype=np.float32)
    for r in range(64):
        half += rows[:, :, r]
    want = _interleaved(half[:, 0] + half[:, 1], n)
    assert np.array_equal(qbar, want), np.abs(qbar - want).max()
