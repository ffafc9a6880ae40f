"""Gate parameter gradients in the launch that adds the pooled query's share: not a chain where the sequence is short."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d,m,n,name", [("bf16", 128, 128, 64, "wersa_add_pooled"), ("bf16", 128, 128, 256, "wersa_add_pooled"),
                                              ("f32", 64, 128, 64, "split_filter_bwd")])
def test_many_parameters_on_a_short_sequence(dtype, d, m, n, name):
    """64 heads, L 6: 115 to 227 blocks of 256 gradients, each a chain of dependent loads over the batch.  Side by side on 256 compute units
    they take a few microseconds of the launch; one after the other on its 1 to 4 workgroups per row they took that many times as long.  The
    launch with the gradients is compared with the one without (whose blocks return at once), the shortest of ten each."""
    import torch
    from paper_2507_08637_amd import binding
    H, L = 64, 6
    g = torch.Generator(device="cuda").manual_seed(d + n)

    def normal(*s):
        return torch.randn(s, generator=g, device="cuda")

    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    q, k, v, dout = (normal(2, H, n, d).to(dt) for _ in range(4))
    par = (normal(d, m).to(dt), torch.ones(1, device="cuda"), normal(H, L + 1, d) / d ** 0.5, normal(H, L + 1), 1 + 0.1 * normal(L + 1))
    out, saved = binding.wersa_forward(q, k, v, *par, L)
    shortest = {}
    for grads in (True, False):
        times = []
        for _ in range(10):
            binding.wersa_profile_enable(True, only=name)
            binding.wersa_backward(q, k, v, *par, out, dout, saved, L, param_grads=grads)
            ms, launches = binding.wersa_profile_collect()[name]
            assert launches == 1
            times.append(1e3 * ms)
        binding.wersa_profile_enable(False)
        shortest[grads] = min(times)
    print((dtype, d, n), {x: f"{t:.1f} us" for x, t in shortest.items()}, flush=True)
    assert shortest[True] < shortest[False] + 15
