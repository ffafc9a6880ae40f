"""Which kernels a call launches, on a stand-in for the HIP runtime: the rules of the dispatch, and what becomes of a runtime call that fails."""
import pytest

from tests.launches import launches


def desc(slices, n, d, m, L=4, bf16=True, **kw):
    from paper_2507_08637_amd.binding import WersaDesc
    return WersaDesc(1, slices, n, d, L, m, int(bf16), 1e-6, 1e-6, slices * n * d, n * d, d, kw.get("flags", 0))


def kernels(what, *a, **kw):
    (status, error, found), = launches([(what, desc(*a, **kw))])
    assert (status, error) == (0, 0)
    return found


@pytest.mark.parametrize("what,lds,memory", [("forward", "deep_addend_kernel<1>", "deep_addend_kernel<0>"), ("backward", "deep_bwd_kernel<1>", "deep_bwd_kernel<0>")])
def test_pyramids_go_to_memory_where_the_runtime_refuses_the_lds(what, lds, memory):
    """The refused attribute is not an error of the call."""
    call = [(what, desc(2, 60000, 32, 64, L=10, bf16=False))]
    (good,), (bad,) = launches(call), launches(call, fail_attributes=True)
    assert good[:2] == bad[:2] == (0, 0)
    names = [k[0] for k in good[2]]
    assert lds in names and memory not in names
    assert [k[0] for k in bad[2]] == [memory if x == lds else x for x in names]


@pytest.mark.parametrize("slices,n,m,apart", [
    (8, 4096, 256, False), (512, 64, 256, False), (1023, 64, 128, False), (1023, 64, 256, False), (128, 64, 1024, False), (129, 64, 1024, True),
    (768, 256, 512, False), (769, 256, 512, True), (128, 64, 2048, True), (64, 64, 4096, True), (32, 64, 4096, False), (170, 64, 384, False), (171, 64, 384, True)])
def test_gate_has_a_launch_of_its_own_where_many_workgroups_would_form_it_again(slices, n, m, apart):
    names = [k[0] for k in kernels("forward", slices, n, 64, m)]
    assert ("gate_fwd_kernel" in names) == apart


@pytest.mark.parametrize("slices,n,waves", [
    (1, 1, 8), (1, 256, 8), (1, 257, 4), (8, 200, 8), (96, 256, 8), (96, 257, 4), (96, 512, 4), (192, 256, 8), (20, 3000, 4), (128, 320, 4), (1, 65536, 4), (85, 769, 8), (129, 320, 8), (8, 8193, 8), (500, 64, 8), (500, 320, 8), (8, 65536, 8)])
def test_rows_kernels_have_four_waves_where_that_gives_more_workgroups(slices, n, waves):
    for what, names in (("forward", ["rows_kernel"]), ("backward", ["masked_rows_kernel"] * 2 + ["rows_kernel"])):
        found = [(name.split("<")[0], threads) for name, _, threads, _ in kernels(what, slices, n, 64, 256) if "rows_kernel<" in name]
        assert sorted(found) == [(name, 64 * waves) for name in names]


@pytest.mark.parametrize("kw", [dict(L=7), dict(flags=8)])
def test_rows_kernels_with_deep_levels_or_layernorm_have_eight_waves(kw):
    for what in ("forward", "backward"):
        assert {threads for name, _, threads, _ in kernels(what, 4, 1000, 64, 256, **kw) if "rows_kernel<" in name} == {512}


@pytest.mark.parametrize("slices,n,d,m,L,chunks", [
    (800, 4720, 64, 48, 2, 3), (893, 1163, 48, 176, 5, 3), (1, 1024, 64, 64, 3, 16), (1, 40, 16, 16, 1, 1), (3, 1000, 32, 64, 8, 16)])
def test_every_workgroup_of_the_pooling_launch_has_something_to_do(slices, n, d, m, L, chunks):
    """The chunks of all slices, the packing of Omega once (64 pieces per 32 features and operand tile, 256 to a workgroup) and one that clears."""
    dh = next(x for x in (16, 32, 64, 128) if d <= x)
    pieces = (m + 31) // 32 * 64 * (dh // 16 + 2 * max(1, dh // 32))
    grid, = (grid for name, grid, _, _ in kernels("forward", slices, n, d, m, L, bf16=False) if name.startswith("pool_kernel"))
    assert grid == ((pieces + 255) // 256 + 1 + chunks * slices, 1, 2 if L > 6 else 1)


@pytest.mark.parametrize("slices,n,d,m,bf16,splits", [
    (1, 1024, 64, 64, False, 8),      # four token tiles: sixteen shares (two: 32)
    (4, 1000, 128, 256, False, 16),   # two tiles
    (13, 490, 64, 128, False, 8),     # two tiles: sixteen shares
    (160, 185, 64, 64, False, 1),     # four tiles would be 320 workgroups
    (120, 382, 96, 128, True, 2),     # 360
    (54, 961, 64, 128, False, 4),     # 432
    (26, 715, 32, 32, False, 6),      # head dimension 32: four at least
    (16, 182, 48, 32, True, 1),       # six shares from two
    (6, 89, 48, 384, False, 1),       # four shares from two
    (38, 87, 64, 256, False, 2),      # two shares from one tile's worth
    (9, 3940, 16, 64, True, 16),      # one-term operands: eight at least
    (2, 2882, 32, 64, True, 12)])
def test_contraction_is_split_finer_within_one_round(slices, n, d, m, bf16, splits):
    for what in ("forward", "backward"):
        (name, grid, _, _), = (k for k in kernels(what, slices, n, d, m, bf16=bf16) if k[0].startswith("contract_kernel"))
        assert grid[0] == splits and grid[2] == slices


@pytest.mark.parametrize("slices,n,d,apart", [
    (1, 1024, 64, False), (1, 131072, 64, True), (10, 4000, 32, False), (22, 1984, 64, False), (22, 1985, 64, True), (22, 192, 128, False), (4, 512, 128, False),
    (4, 513, 128, True), (6, 2190, 96, True), (85, 256, 128, False), (86, 256, 128, True)])
def test_gate_of_the_split_path_has_a_launch_of_its_own(slices, n, d, apart):
    """More than 2048 packing workgroups of 4096 elements, or above head dimension 64 more than eight chunks of partial sums."""
    names = [k[0] for k in kernels("forward", slices, n, d, 96, L=3, bf16=False)]
    assert ("gate_fwd_kernel" in names) == apart
