"""Split path (float32 arithmetic on the bf16 matrix cores: three bf16 terms per float32 operand) at the sizes
where its kernels change shape: head dimensions padded to 16, 32, 64, 128; feature counts that are not whole
32-feature tiles, or an odd number of them; token counts around the 32- and 64-row tiles and the
4096-element workgroups; few rows (2-wave workgroups) and many (4 waves, 8 at head dimension 64); rows that are not 16-byte
aligned."""
import numpy as np
import pytest

from tests import helpers as hp
from paper_2507_08637_amd import workloads

pytestmark = pytest.mark.gpu

# O, S, z and D against float64: operands exact to 2^-24 and accumulators rounded at most some thousand times, which
# adds up like a random walk: 2^-24 * sqrt(1000) = 1.9e-6.
SUMS = 2e-6


def _grad_tol(cfg):
    """The float32 bar of the library, 1e-4, unless pre-activations within a few rounding errors of zero (a share of
    about 2e-7 of them) are to be expected in a problem of this size: each that takes the other side of the ReLU's
    step changes its row by one of about m / 2 terms, a share 2 / m of the row's squared norm."""
    if cfg["dtype"] == "bf16":
        return 2e-2
    rows = cfg["B"] * cfg["H"] * cfg["n"]
    flips = 2e-7 * rows * cfg["m"]
    return 1e-4 if flips < 0.1 else max(1e-4, ((4 + 4 * flips) * (2 / cfg["m"]) / rows) ** 0.5)


SHAPES = [
    dict(B=1, H=1, n=65, d=16, L=2, m=16),       # half a feature tile; one row past a 64-row block
    dict(B=2, H=3, n=257, d=16, L=5, m=544),     # 17 feature tiles: every wave of the contraction takes the same one; one row past 256
    dict(B=1, H=2, n=31, d=32, L=1, m=96),       # less than one token tile; three feature tiles
    dict(B=1, H=2, n=129, d=48, L=6, m=64),      # columns padded to 64, two feature tiles
    dict(B=2, H=1, n=2300, d=64, L=9, m=256),    # levels above one tile, ragged
    dict(B=1, H=2, n=97, d=112, L=3, m=160),     # columns padded to 128, five feature tiles
    dict(B=1, H=1, n=700, d=128, L=7, m=48),
    dict(B=16, H=16, n=520, d=16, L=3, m=64),    # 4-wave workgroups, the last one partly idle
    dict(B=16, H=16, n=260, d=32, L=4, m=128),
    dict(B=16, H=16, n=200, d=64, L=0, m=32),
]


def _check(res, ref, fwd, cfg):
    grads = _grad_tol(cfg)
    for k in ("S", "z", "D"):
        assert hp.rel_err(res["saved"][k], fwd[k].reshape(res["saved"][k].shape)) < SUMS, k
    assert hp.rel_err(res["O"], ref["O"]) < (SUMS if cfg["dtype"] == "f32" else 4e-3), "O"   # bf16: rounded once, by 2^-9 at most
    for k in ("dQ", "dK", "dV") + (("dWg", "dbg") if cfg["L"] and cfg["dtype"] == "f32" else ()):
        assert hp.rel_err(res[k], ref[k]) < grads, k


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "B{B}H{H}n{n}d{d}L{L}m{m}".format(**s))
def test_split_path_shapes(shape, dtype):
    cfg = dict(shape, dtype=dtype, flavour="plain", seed_base=5100, q_mean=0.5)
    p = workloads.make_inputs(**cfg)
    res = hp.gpu_forward_backward(p, cfg, flags=1)
    _check(res, hp.oracle_backward(p, cfg), hp.oracle_forward(p, cfg), cfg)


@pytest.mark.parametrize("L", [3, 8])
def test_few_rows_many_features_keep_the_generic_kernels(L):
    """The shape class that fits wersa_forward_static's scratch on the generic kernels alone: forward and backward
    meet the same bars, and the call without workspace gives the same bits as the one with."""
    import torch
    from paper_2507_08637_amd import binding
    cfg = dict(B=1, H=32, n=64, d=128, L=L, m=1024, dtype="f32", flavour="plain", seed_base=5300, q_mean=0.5)
    p = workloads.make_inputs(**cfg)
    res = hp.gpu_forward_backward(p, cfg, flags=1)
    _check(res, hp.oracle_backward(p, cfg), hp.oracle_forward(p, cfg), cfg)
    t = hp.to_device(p, "f32")
    args = (t["Q"], t["K"], t["V"], t["Omega"], t["sigma"], t["Wg"], t["bg"], t["omega"], L)
    ref, saved = binding.wersa_forward(*args)
    out = torch.empty_like(ref)
    binding.wersa_forward_static(*args, out, torch.empty_like(saved))
    assert torch.equal(out, ref)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_split_path_rows_off_16_byte_alignment(dtype):
    """A row stride of d + 1 elements: every load of the packing kernels falls back to single elements, same bits."""
    import torch
    from paper_2507_08637_amd import binding
    cfg = dict(B=1, H=2, n=200, d=32, L=3, m=64, dtype=dtype, flavour="plain", seed_base=5200, q_mean=0.5)
    t = hp.to_device(workloads.make_inputs(**cfg), dtype)
    outs = []
    for pad in (0, 1):
        def lay(x):
            y = torch.zeros(*x.shape[:3], x.shape[3] + pad, dtype=x.dtype, device=x.device)[..., :x.shape[3]]
            return y.copy_(x)
        q, k, v, do = (lay(t[name]) for name in ("Q", "K", "V", "dO"))
        par = (t["Omega"], t["sigma"], t["Wg"], t["bg"], t["omega"])
        out, saved = binding.wersa_forward(q, k, v, *par, cfg["L"], flags=1)
        g = binding.wersa_backward(q, k, v, *par, out, do, saved, cfg["L"], flags=1)
        outs.append([out, g["dq"], g["dk"], g["dv"], g["dgate_w"]])
    for a, b in zip(*outs):
        assert torch.equal(a, b)


@pytest.mark.parametrize("n,d,m,bound", [
    # long chains over the features (D, O): sixteen features, eight of these, sixteen of those for D; for O one rounding of
    # its accumulator per 16 features
    (2048, 32, 4096, dict(S=1.5e-7, z=1.2e-7, D=1.5e-7, O=4.5e-7)),
    (2048, 16, 4096, dict(S=1.5e-7, z=1.2e-7, D=1.5e-7, O=4.5e-7)),
    # and over the tokens (S, z): hundreds of shares
    (100000, 64, 128, dict(S=1.4e-7, z=1.4e-7, D=1.4e-7, O=1.3e-7)),
])
def test_sums_stay_close_to_float64(n, d, m, bound):
    """n additions of like terms one after the other are off by about 2.5e-8 sqrt(n / 3), so the bounds hold chains of a few
    ten at the most; the kernels that wrote every feature matrix to memory met D 1.5e-7, O 6.7e-7, z 2.5e-7 here, one chain
    for each sum D 3.4e-7, O 6.9e-7, S and z 4e-7.  Medians over seven inputs."""
    import torch
    from paper_2507_08637_amd import binding
    L, errs = 2, {}
    for seed in range(7):
        g = torch.Generator(device="cuda").manual_seed(seed)

        def normal(*s):
            return torch.randn(s, generator=g, device="cuda")

        wave = torch.sin(torch.arange(n, device="cuda") / 40.0)[:, None]
        q, k, v = (normal(n, d) * s + a * wave + c for s, a, c in ((1, 0.7, 0.2), (1, 0.7, 0.2), (0.3, 1, 1)))
        omega, sigma, gw, gb = normal(d, m), torch.ones(1, device="cuda"), normal(1, L + 1, d) / d ** 0.5, 0.5 * normal(1, L + 1)
        sw = 1 + 0.1 * normal(L + 1)
        qkv = [x[None, None] for x in (q, k, v)]
        out, saved = binding.wersa_forward(*qkv, omega, sigma, gw, gb, sw, L)
        got = binding.saved_views(binding.make_desc(qkv[0], L, m), saved)
        # (only what the sums are made of: the filter as the library computed it)
        F = got["F"][0].double()

        def filtered(x):
            y = F[0] * x
            for lvl in range(1, L + 1):
                pad = -n % (1 << lvl)
                z = torch.cat([x, x.new_zeros(pad, d)]).view(-1, 1 << lvl, d).mean(1, keepdim=True)
                y = y + (F[lvl] - F[lvl - 1]) * z.expand(-1, 1 << lvl, -1).reshape(-1, d)[:n]
            return y

        Q, K = filtered(q.double()), filtered(k.double())
        c = 1 / m ** 0.5
        pk, pq = torch.relu(K @ omega.double()) * c, torch.relu(Q @ omega.double()) * c
        S, z = pk.t() @ v.double(), pk.sum(0)
        D = pq @ z + 1e-6
        O = pq @ S / D[:, None]
        ref = dict(S=S, z=z, D=D, O=O)
        res = dict(S=got["S"][0], z=got["z"][0], D=got["D"][0], O=out[0, 0])
        for name, r in ref.items():
            errs.setdefault(name, []).append(float((res[name].double() - r).norm() / r.norm()))
    med = {name: sorted(e)[3] for name, e in errs.items()}
    print((n, d, m), {name: f"{e:.2e}" for name, e in med.items()}, flush=True)
    assert all(med[name] < b for name, b in bound.items()), med


NONFINITE = [("bf16", 16, 96, 2), ("bf16", 32, 64, 3), ("f32", 16, 64, 0), ("f32", 32, 96, 2), ("f32", 64, 64, 5), ("f32", 128, 64, 3)]


@pytest.mark.parametrize("bad", [float("nan"), -float("nan"), float("inf")], ids=["nan", "minus_nan", "inf"])
@pytest.mark.parametrize("dtype,d,m,L", NONFINITE)
def test_where_a_value_that_is_not_finite_goes(dtype, d, m, L, bad):
    """The ReLU of a NaN of either sign is 0, in the features and in their derivative, and nothing crosses to rows outside the
    2^L rows of the filter's block, to other columns of V and dO or to other slices."""
    import struct
    import torch
    from paper_2507_08637_amd import binding
    B, H, n, t, j = 1, 2, 200, 77, 5
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    if bad != bad:   # the sign has to reach the tensor
        bits = torch.tensor([-0x400000 if struct.pack(">d", bad)[0] & 0x80 else 0x7fc00000], dtype=torch.int32)
        value = bits.view(torch.float32).to(tdt).cuda()[0]
    else:
        value = bad
    g = torch.Generator(device="cuda").manual_seed(d + m)

    def normal(*s):
        return torch.randn(s, generator=g, device="cuda")

    clean = {k: normal(B, H, n, d).to(tdt) for k in ("q", "k", "v", "do")}
    par = (normal(d, m).to(tdt), torch.ones(1, device="cuda"), normal(H, L + 1, d) / d ** 0.5, normal(H, L + 1),
           1 + 0.1 * normal(L + 1))

    def run(where):
        x = {k: v.clone() for k, v in clean.items()}
        if where:
            x[where][0, 0, t, j] = value
        out, saved = binding.wersa_forward(x["q"], x["k"], x["v"], *par, L, flags=1)
        g = binding.wersa_backward(x["q"], x["k"], x["v"], *par, out, x["do"], saved, L, flags=1)
        sv = binding.saved_views(binding.make_desc(x["q"], L, m, flags=1), saved)
        return dict(g, out=out, **{k: v.clone() for k, v in sv.items()})

    ref = run(None)
    for where in clean:
        got = run(where)
        for name in ("out", "dq", "dk", "dv"):   # the other head
            assert torch.equal(got[name][0, 1], ref[name][0, 1]), (where, name)
        o, dv = got["out"][0, 0], got["dv"][0, 0]
        rest = [c for c in range(d) if c != j]
        if where == "q" and bad != bad:   # the pooled query makes every filter coefficient NaN: no feature is left
            assert bool((o == 0).all()) and bool((dv == 0).all()) and bool((got["S"][0] == 0).all())
        elif where == "k" and bad != bad:   # the rows of its block have no features
            lo = t >> L << L
            F = ref["F"][0].double()
            K = clean["k"][0, 0].double()
            x = F[0] * K
            for lvl in range(1, L + 1):
                z = K[:n >> L << L].view(-1, 1 << lvl, d).mean(1, keepdim=True).expand(-1, 1 << lvl, -1).reshape(-1, d)
                x[:z.shape[0]] += (F[lvl] - F[lvl - 1]) * z
                x[z.shape[0]:] = 0   # (an incomplete last block: left out of the comparison below)
            whole = (n >> L << L) == n
            phi = torch.relu(x @ par[0].double()) / m ** 0.5
            phi[lo:lo + (1 << L)] = 0
            if whole:
                z = got["z"][0].double()
                assert float((z - phi.sum(0)).norm() / z.norm()) < 1e-5
            assert bool(torch.isfinite(o.float()).all())
        elif where == "v":
            assert not bool(torch.isfinite(o[:, j].float()).any())
            assert torch.equal(o[:, rest], ref["out"][0, 0][:, rest])
        elif where == "do":
            assert not bool(torch.isfinite(dv[:, j].float()).any())
            assert torch.equal(dv[:, rest], ref["dv"][0, 0][:, rest])


@pytest.mark.parametrize("d,m,n", [(16, 96, 200), (32, 64, 500), (64, 96, 330), (128, 64, 200)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_magnitudes_far_apart(dtype, d, m, n):
    """Tokens up to 2^20 apart in Q, K and V, columns of V and features of Omega 2^8 apart, dO 2^30 above the rest.  Every row and
    column of S, every feature of z, every row of O and every column of dV on its own: the worst of 2^-24 per factor and term grows
    with the sum's length as sqrt(n + m) at most, times 4 for cancellation; bf16: the output's rounding.  dQ and dK as a whole here,
    element by element in test_columns_of_unlike_size."""
    import torch
    from paper_2507_08637_amd import binding
    g = torch.Generator(device="cuda").manual_seed(d + n)
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16

    def normal(*s):
        return torch.randn(s, generator=g, device="cuda")

    def spread(lo, hi, *s):
        return 2.0 ** torch.randint(lo, hi + 1, s, generator=g, device="cuda").float()

    tile = torch.arange(n, device="cuda") // 32
    steps = spread(-10, 10, int(tile[-1]) + 1)
    q = (normal(n, d) + 0.3) * spread(-10, 10, n, 1)
    k = (normal(n, d) + 0.3) * spread(-3, 3, n, 1) * 2.0 ** -20
    v = (0.3 * normal(n, d) + 1) * steps[tile][:, None] * spread(-4, 4, d)
    do = (0.3 * normal(n, d) + 0.5) * 2.0 ** 30
    q, k, v, do = (x.to(tdt)[None, None] for x in (q, k, v, do))
    omega = (normal(d, m) * spread(-4, 4, m)).to(tdt)
    par = (omega, torch.ones(1, device="cuda"), torch.zeros(1, 1, d, device="cuda"), torch.zeros(1, 1, device="cuda"),
           2 * torch.ones(1, device="cuda"))   # no levels, F = 1: rows keep their own magnitudes
    out, saved = binding.wersa_forward(q, k, v, *par, 0, eps=1e-30, flags=1)
    got = binding.wersa_backward(q, k, v, *par, out, do, saved, 0, eps=1e-30, flags=1)
    sv = binding.saved_views(binding.make_desc(q, 0, m, 1e-30, 1e-6, 1), saved)
    Q, K, V = (x[0, 0].double().requires_grad_() for x in (q, k, v))
    phi = [torch.relu(x @ omega.double()) / m ** 0.5 for x in (Q, K)]
    S, z = phi[1].t() @ V, phi[1].sum(0)
    O = phi[0] @ S / (phi[0] @ z + 1e-30)[:, None]
    gQ, gK, gV = torch.autograd.grad(O, (Q, K, V), do[0, 0].double())

    def worst(a, r, dim):
        a, r = a.double(), r.detach()
        return float(((a - r).norm(dim=dim) / r.norm(dim=dim).clamp_min(1e-300)).max())

    bound = 4 * 2.0 ** -24 * (n + m) ** 0.5
    errs = dict(S=worst(sv["S"][0], S, 1), S_columns=worst(sv["S"][0], S, 0), z=worst(sv["z"][0][:, None], z[:, None], 1),
                O=worst(out[0, 0], O, 0), dV=worst(got["dv"][0, 0], gV, 0))
    print(dtype, d, {k: f"{e:.1e}" for k, e in errs.items()}, f"bound {bound:.1e}", flush=True)
    for name, e in errs.items():
        assert e < bound + (2.0 ** -8 if dtype == "bf16" and name in ("O", "dV") else 0), (name, errs)
    if dtype == "f32":   # (dQ and dK through cancellation: their size, and that nothing overflowed on the way)
        for a, r in ((got["dq"], gQ), (got["dk"], gK)):
            assert bool(torch.isfinite(a).all()) and float((a[0, 0].double() - r).norm() / r.norm()) < 1e-4


@pytest.mark.parametrize("d,m,n", [(16, 64, 8200), (32, 64, 4100), (64, 64, 8200), (128, 96, 4100)])   # 33 to 129 shares of the tokens
@pytest.mark.parametrize("kind,k", [("columns", 24), ("columns", 40), ("classes", 40), ("projection", 40)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_columns_of_unlike_size(dtype, kind, k, d, m, n):
    """Every operand has float32's exponent range element by element, so no element of a result loses to a larger one beside it.
    columns: half of the columns of V times 2^-k, of dO times 2^k, so both halves have the same weight in dPhi.
    classes: the small columns of one half of the tokens are the large ones of the other half, and no feature sees both, so no power
    of two per row and column makes the tokens alike.
    projection: half of the columns of Q and K times 2^-k, of Omega's rows times 2^k.
    Each element is held to its own sum of absolute values: 2^-24 for each rounding on its way, all of them the same way round.
    Accumulators: d / 16 steps (projection, dPhi), 2 * 8 of a share, 129 shares at most, m / 16, six products each (three of them below 2^-16);
    operands and scalings 20.  bf16 storage: O, which the backward reads, and the result are rounded by 2^-9 each; the rounding of O
    comes back in dD, and through dz in dK: 2^-7.  Rows of dQ and dK with a pre-activation within 2^-16 of its own sum of absolute
    values are left out: it may fall on the other side of the ReLU's step."""
    import torch
    from paper_2507_08637_amd import binding
    g = torch.Generator(device="cuda").manual_seed(d + n + k)
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16

    def normal(*s):
        return torch.randn(s, generator=g, device="cuda")

    q, k_, v, do = normal(n, d) + 0.3, normal(n, d) + 0.3, 0.3 * normal(n, d) + 1, 0.3 * normal(n, d) + 0.5
    omega = normal(d, m)
    half = torch.arange(d, device="cuda") % 2 == 0
    if kind == "projection":
        q[:, half] *= 2.0 ** -k
        k_[:, half] *= 2.0 ** -k
        omega[half] *= 2.0 ** k
    else:
        small = half.expand(n, d)
        if kind == "classes":
            second = torch.arange(n, device="cuda") % 2 == 1
            small = small ^ second[:, None]
            for x in (q, k_):
                x *= 0.2
                x[:, 0] = torch.where(second, -30.0, 30.0)
            omega[0] = torch.where(torch.arange(m, device="cuda") % 2 == 1, -1.0, 1.0)
        v[small] *= 2.0 ** -k
        do[small] *= 2.0 ** k
    q, k_, v, do = (x.to(tdt)[None, None] for x in (q, k_, v, do))
    omega = omega.to(tdt)
    par = (omega, torch.ones(1, device="cuda"), torch.zeros(1, 1, d, device="cuda"), torch.zeros(1, 1, device="cuda"),
           2 * torch.ones(1, device="cuda"))   # no levels, F = 1
    out, saved = binding.wersa_forward(q, k_, v, *par, 0, eps=1e-30, flags=1)
    got = binding.wersa_backward(q, k_, v, *par, out, do, saved, 0, eps=1e-30, flags=1)
    sv = binding.saved_views(binding.make_desc(q, 0, m, 1e-30, 1e-6, 1), saved)

    # the exact values and, with the same products of absolute values, what each element is a sum of
    def chain(sign):
        f = (lambda x: x) if sign else torch.abs
        Q, K, V, dO, W = (f(x.double().reshape(-1, x.shape[-1])) for x in (q, k_, v, do, omega))
        phi = [(X @ W / m ** 0.5) * on for X, on in ((Q, on_q), (K, on_k))]
        S, z = phi[1].t() @ V, phi[1].sum(0)
        D = phi[0] @ z if sign else real["D"]
        O = phi[0] @ S / D[:, None]
        dN, dD = dO / D[:, None], f(-(dO * O).sum(1) / D)
        dS, dz = phi[0].t() @ dN, phi[0].t() @ dD
        dQ = ((dN @ S.t() + dD[:, None] * z) * on_q) @ W.t() / m ** 0.5
        dK = ((V @ dS.t() + dz) * on_k) @ W.t() / m ** 0.5
        return dict(S=S, z=z, D=D, O=O, dq=dQ, dk=dK, dv=phi[1] @ dS)

    W = omega.double()
    R = [x[0, 0].double() @ W for x in (q, k_)]
    on_q, on_k = ((r > 0).double() for r in R)
    sure = [(r.abs() > 2.0 ** -16 * (x[0, 0].double().abs() @ W.abs())).all(1) for r, x in zip(R, (q, k_))]
    real = chain(True)
    size = chain(False)
    roundings = 6 * (2 * (d // 16) + 2 * 8 + m // 16) + 129 + 20
    bound = roundings * 2.0 ** -24
    errs = {}
    for name, a in dict(S=sv["S"][0], z=sv["z"][0], O=out[0, 0], dq=got["dq"][0, 0], dk=got["dk"][0, 0], dv=got["dv"][0, 0]).items():
        assert bool(torch.isfinite(a).all()), name
        e = (a.double() - real[name]).abs() / size[name]
        if name in ("dq", "dk"):
            keep = sure[name == "dk"]
            assert int(keep.sum()) > n // 2
            e = e[keep]
        errs[name] = float(e.max())
    print(dtype, kind, k, d, {x: f"{e:.1e}" for x, e in errs.items()}, f"bound {bound:.1e}", flush=True)
    for name, e in errs.items():
        assert e < bound + (2.0 ** -7 if dtype == "bf16" and name not in ("S", "z") else 0), (name, errs)


@pytest.mark.parametrize("d", [16, 32, 64, 128])
def test_sums_over_many_features(d):
    """Sums over 4096 features are taken in parts (128 features, 32 from d 64 on), so their error does not grow with every product:
    32 or 128 roundings of the total, 2^-24 of it at most and of random sign, add up to 2^-24 * sqrt(128 / 3) / 2 = 2e-7; the
    parts' own roundings (24 products each, 48 or more parts) and the operands are below a third of it, D and the rest of O's way
    2^-24 twice.  Together 3e-7; in one accumulator: O 3.4e-7 and dV 5.9e-7 at 2048 tokens, d 32.  (d 64: dV in one accumulator.)"""
    cfg = dict(B=1, H=1, n=512, d=d, L=2, m=4096, dtype="f32", flavour="plain", seed_base=6200 + d, q_mean=0.5)
    p = workloads.make_inputs(**cfg)
    res = hp.gpu_forward_backward(p, cfg, flags=1)
    ref = hp.oracle_backward(p, cfg)
    errs = {k: hp.rel_err(res[k], ref[k]) for k in ("O", "dV")}
    print(cfg, {k: f"{e:.2e}" for k, e in errs.items()}, flush=True)
    assert errs["O"] < 3e-7 and (d == 64 or errs["dV"] < 3e-7), errs
