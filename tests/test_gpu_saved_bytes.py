"""The split path's `saved`: every byte is written by the forward, so what the memory held before does not show in it.  Shapes
with and without the packed Q_F and K_F, sections of lengths that are no multiple of 64, levels above 6, options."""
import pytest

from paper_2507_08637_amd import workloads
from tests import helpers as hp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,H,n,d,m,L,flags", [
    ("f32", 1, 1024, 64, 64, 3, 0), ("f32", 3, 1000, 32, 48, 7, 0), ("bf16", 2, 777, 16, 48, 9, 0), ("f32", 1, 5000, 80, 48, 8, 1),
    ("bf16", 2, 3001, 32, 80, 4, 1), ("bf16", 6, 120001, 16, 32, 3, 0), ("f32", 2, 40000, 128, 32, 3, 0)])
def test_saved_does_not_depend_on_the_memory(dtype, H, n, d, m, L, flags):
    import torch
    from paper_2507_08637_amd import binding
    p = workloads.make_inputs(B=1, H=H, n=n, d=d, L=L, m=m, dtype=dtype, flavour="plain", seed_base=7600, q_mean=0.4)
    t = hp.to_device(p, dtype)
    args = (t["Q"], t["K"], t["V"], t["Omega"], t["sigma"], t["Wg"], t["bg"], t["omega"], L)
    _, saved = binding.wersa_forward(*args, flags=flags)
    results = []
    for word in (0, -1):   # (-1: NaN in float32 and in bf16)
        buf = torch.full((saved.numel(),), word, dtype=torch.int32, device="cuda")
        binding.wersa_forward(*args, saved=buf.view(torch.float32), flags=flags)
        results.append(buf)
    assert torch.equal(*results)
