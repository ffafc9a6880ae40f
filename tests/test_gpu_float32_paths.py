"""The two sets of kernels with float32 arithmetic, with the options of Algorithm 1 and the shapes that change their form,
against the oracle: the split path at every padded head dimension (one-term bf16 operands, odd numbers of feature
tiles over two random matrices, LayerNorm), the generic kernels at head dimensions above 128, with few rows, and
with transforms whose second stage has several tiles.  Which of the two a descriptor takes is told from `saved` (the
split path keeps operands of Omega there)."""
import ctypes

import numpy as np
import pytest

from paper_2507_08637_amd import workloads
from tests import helpers as hp

pytestmark = pytest.mark.gpu

EPS = 1e-3   # the bandwidth's gradient is of its order


def _path(cfg, flags):
    from paper_2507_08637_amd import binding
    H, n, d, m, nb = cfg["H"], cfg["n"], cfg["d"], cfg["m"], cfg["L"] + 1
    desc = binding.WersaDesc(cfg["B"], H, n, d, cfg["L"], m, 0 if cfg["dtype"] == "f32" else 1, EPS, 1e-6, H * n * d, n * d, d, flags)
    lib = binding.load_library()
    assert lib.wersa_selected_path(ctypes.byref(desc)) == 0
    sl = cfg["B"] * H
    plain = sum((k + 63) // 64 * 64 for k in (sl * m * d, sl * m, sl * d, sl * nb, sl * nb, sl * n)) * 4
    return "generic" if lib.wersa_saved_bytes(ctypes.byref(desc)) == plain else "split"


def _check(cfg, flags, few_rows=False):
    """float32: 1e-4 on O and its gradients as everywhere, the sums in `saved` 5e-6; bf16: 2e-2.  The gate's gradients to the same
    share of their un-cancelled magnitude (helpers.gate_grad_scales).  With few rows dQ is the small difference of large terms
    (the rows of O differ little), which bf16 rounding of O leaves nothing of: not checked there in bf16."""
    p = workloads.make_inputs(**cfg)
    f32, pooled, ln = cfg["dtype"] == "f32", bool(flags & 4), bool(flags & 8)
    if flags & 2:
        omk = np.random.default_rng(cfg["seed_base"] + 99).standard_normal(p["Omega"].shape, dtype=np.float32)
        p["OmegaK"] = omk if f32 else workloads.round_to_bf16(omk)
    res = hp.gpu_forward_backward(p, cfg, eps=EPS, flags=flags)
    ref = hp.oracle_backward(p, cfg, eps=EPS, pooled=pooled, layernorm=ln)
    if not pooled:   # (the oracle's forward on its own has the per-head gate)
        fwd = hp.oracle_forward(p, cfg, eps=EPS, layernorm=ln)
        for k in ("S", "z", "D"):
            assert hp.rel_err(res["saved"][k], fwd[k].reshape(res["saved"][k].shape)) < 5e-6, k
    errs = {k: hp.rel_err(res[k], ref[k]) for k in ("O", "dQ", "dK", "dV")}
    scales = hp.gate_grad_scales(p, cfg, eps=EPS, layernorm=ln)
    heads = cfg["H"] if pooled else 1   # (pooled: every head's logits get the sum over the heads)
    gate = {k: hp.scaled_err(res[k], ref[k], scales[k]) / heads for k in ("dWg", "dbg", "domega")}
    sig = abs(float(res["dsigma"].cpu()) - ref["dsigma"]) / abs(ref["dsigma"])
    print(cfg, flags, {k: f"{v:.1e}" for k, v in dict(errs, **gate, dsigma=sig).items()}, flush=True)
    if few_rows and not f32:
        errs.pop("dQ")
        gate = {}
    assert all(v < (1e-4 if f32 else 2e-2) for v in dict(errs, **gate).values()), (errs, gate)
    assert sig < (1e-3 if f32 else 2e-2)


OPTIONS = [0, 2, 4, 8, 14]


@pytest.mark.parametrize("flags", OPTIONS)
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d,m,n,L", [(16, 96, 200, 2), (32, 96, 130, 3), (48, 80, 300, 8), (80, 48, 150, 4), (128, 160, 100, 5)])
def test_options_on_the_split_path(d, m, n, L, dtype, flags):
    cfg = dict(B=2, H=3, n=n, d=d, L=L, m=m, dtype=dtype, flavour="plain", seed_base=7100, q_mean=0.4)
    flags |= 1 if d == 128 else 0
    assert _path(cfg, flags) == "split"
    _check(cfg, flags)


@pytest.mark.parametrize("flags", OPTIONS)
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("H,d,m,n,L", [(3, 160, 48, 200, 3), (2, 256, 80, 130, 7), (1, 144, 16, 4500, 9),   # above 128; 71 tiles in the second stage
                                       (2, 128, 1024, 20, 2), (1, 80, 1024, 3, 1)])                          # few rows
def test_options_on_the_generic_kernels(H, d, m, n, L, dtype, flags):
    cfg = dict(B=2 if n < 1000 else 1, H=H, n=n, d=d, L=L, m=m, dtype=dtype, flavour="plain", seed_base=7200, q_mean=0.4)
    flags |= 1 if d == 128 else 0
    assert _path(cfg, flags) == "generic"
    _check(cfg, flags, few_rows=n <= 20)


@pytest.mark.parametrize("dtype,H,n,d,m", [("f32", 2, 60000, 64, 48), ("f32", 2, 40000, 128, 32), ("bf16", 6, 120000, 32, 64),
                                           ("bf16", 6, 120001, 16, 32)])
def test_operands_formed_again_by_the_backward(dtype, H, n, d, m):
    """Problems whose Q_F and K_F `saved` does not keep: two backward calls on one forward give the same bits (nothing of
    the first is left in what the second reads), and the gradients meet the bars."""
    import torch
    from paper_2507_08637_amd import binding
    cfg = dict(B=1, H=H, n=n, d=d, L=3, m=m, dtype=dtype, flavour="plain", seed_base=7300, q_mean=0.4)
    assert _path(cfg, 0) == "split"
    p = workloads.make_inputs(**cfg)
    t = hp.to_device(p, dtype)
    par = (t["Omega"], t["sigma"], t["Wg"], t["bg"], t["omega"])
    out, saved = binding.wersa_forward(t["Q"], t["K"], t["V"], *par, 3, eps=EPS)
    assert saved.numel() < H * n * d   # (Q_F and K_F alone would be three times that)
    before = saved.clone()
    a, b = (binding.wersa_backward(t["Q"], t["K"], t["V"], *par, out, t["dO"], saved, 3, eps=EPS) for _ in range(2))
    assert torch.equal(saved, before)
    assert all(torch.equal(a[k], b[k]) for k in a)
    ref = hp.oracle_backward(p, cfg, eps=EPS, slices=[(0, 1)])
    flips = 2e-7 * n * m   # (pre-activations within rounding of zero: see the split path's tests)
    tol = max(1e-4, ((4 + 4 * flips) * (2 / m) / n) ** 0.5) if dtype == "f32" else 2e-2
    for k in ("dQ", "dK", "dV"):
        r = np.asarray(ref[k])
        r = r[0, 1] if r.ndim == 4 else r
        assert hp.rel_err(a[k.lower()][0, 1], r) < tol, k
