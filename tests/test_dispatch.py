"""Which kernel and plan the host layer launches for a call (CPU: the launches
are recorded, not run)."""
import random

import pytest

import dispatch_probe as probe


def log_uniform(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def names(launches):
    return [x.name for x in launches]


def mean_sum(m, n, plan, batch=1):
    """Mean length of an output's running sums, as a share of K."""
    tm, tn, splits, _, whole = plan
    tiles = -(-m // tm) * -(-n // tn) * batch
    return 1.0 if splits == 1 else (whole + (tiles - whole) / splits) / tiles


# ---------------------------------------------------------------------------
# Few rows
# ---------------------------------------------------------------------------

@pytest.mark.parametrize("few,wide,k", [(8, 4096, 4096), (1, 4096, 4096), (16, 4096, 4096), (32, 768, 192),
                                        (8, 2048, 512), (4, 16, 64), (24, 512, 1024)])
@pytest.mark.parametrize("swap", [False, True])
@pytest.mark.parametrize("bf16", [False, True])
def test_few_rows_take_their_kernel(few, wide, k, swap, bf16):
    m, n = (wide, few) if swap else (few, wide)
    got = probe.product(m, n, k, bf16=bf16)
    assert names(got) == ["few rows"]
    # the side with fewer rows is the one held in LDS, also when both are few
    assert bool(got[0].few_rows_of_a) == (m <= n)


@pytest.mark.parametrize("few,wide,k,batch", [
    (32, 32, 65536, 1), (8, 64, 65536, 1), (32, 512, 65536, 1), (16, 16, 16384, 1), (3, 5, 1000000, 1),   # long K
    (32, 32768, 1024, 1), (24, 32768, 256, 1),             # two passes over many rows
    (32, 32, 32, 2048), (8, 64, 32, 2048), (32, 512, 64, 256)])   # many small matrices
def test_few_rows_left_to_the_plan(few, wide, k, batch):
    """Where the few-row kernel leaves the chip idle or works for nothing, the
    product runs its plan (or the small-product kernel)."""
    assert "few rows" not in names(probe.product(few, wide, k, batch))


# ---------------------------------------------------------------------------
# Small products
# ---------------------------------------------------------------------------

@pytest.mark.parametrize("m,n,k,batch", [(256, 256, 256, 1), (512, 512, 256, 1), (1024, 1024, 256, 1), (128, 128, 64, 1),
                                         (197, 64, 197, 16), (256, 256, 640, 1)])
def test_small_products_take_their_kernel(m, n, k, batch):
    assert names(probe.product(m, n, k, batch, tb=False)) == ["small"]


@pytest.mark.parametrize("m,n,k,batch", [(64, 1184, 1696, 1), (96, 288, 1760, 1), (352, 192, 2816, 4),
                                         (256, 256, 2048, 1), (2048, 1024, 256, 1), (128, 128, 4096, 1)])
def test_long_k_small_outputs_keep_their_plan(m, n, k, batch):
    assert names(probe.product(m, n, k, batch, ta=True, tb=False))[0] == "tiled"


@pytest.mark.parametrize("m,n,k,batch,kernel", [
    (32, 32, 32, 2048, "tiled"), (19, 96, 21, 640, "tiled"), (62, 17, 27, 925, "tiled"), (6, 5, 27, 1993, "tiled"),
    (30, 24, 24, 1004, "small"), (7, 22, 24, 1016, "small"), (10, 50, 55, 794, "small"), (8, 5, 48, 1393, "small"),
    (4928, 64, 8, 1, "small"), (29, 24, 4, 300, "small"), (687, 367, 2, 1, "small")])
def test_many_small_matrices_of_short_k(m, n, k, batch, kernel):
    """Up to 32 k steps the small-product kernel's chunk is mostly padding: many
    such matrices keep their plan."""
    assert names(probe.product(m, n, k, batch, tb=False)) == [kernel]


# ---------------------------------------------------------------------------
# Plans
# ---------------------------------------------------------------------------

# Sizes of almost one round of 128 x 128 tiles with long K (and two others)
# whose former plan took most tiles over the whole K and the last 256 in slices:
# (m, n, k) -> that plan's (tiles, whole-K tiles, slices).
NEAR_ONE_ROUND = {(6428, 2368, 3072): (969, 713, 16), (7643, 2043, 2286): (960, 704, 12),
                  (3005, 5230, 10146): (984, 728, 53), (6865, 2208, 3584): (972, 716, 16),
                  (17662, 852, 2400): (966, 710, 15), (14045, 533, 3984): (550, 294, 12), (8400, 945, 2061): (528, 272, 8)}


@pytest.mark.parametrize("size", NEAR_ONE_ROUND, ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("limit", [None, 1 << 30, 256 << 20, 64 << 20])
def test_near_one_round_sums_are_no_longer_than_the_hybrids(size, limit):
    tiles, whole, splits = NEAR_ONE_ROUND[size]
    m, n, k = size
    plan = probe.plan(m, n, k, max_workspace_bytes=limit)
    hybrid_bytes = (tiles - whole) * splits * 128 * 128 * 4
    if limit is None or limit >= hybrid_bytes:
        assert mean_sum(m, n, plan) <= (whole + (tiles - whole) / splits) / tiles, plan


def test_exact_derivative_sums_are_short():
    """K is cut into at least as many slices as doubling gives until tiles of
    128 x 128 times slices reach 1024 (slices of at least four chunks); 56 stand
    for 64, whose reduction adds eights in pairs."""
    rng = random.Random(5)
    sizes = [(1682, 1207, 10324), (12993, 256, 3050), (768, 192, 12608)]
    sizes += [tuple(log_uniform(rng, 16, hi) for hi in (20000, 20000, 30000)) for _ in range(3000)]
    for m, n, k in sizes:
        tiles = -(-m // 128) * -(-n // 128)
        least = 1
        while tiles * least < 1024 and least < 64 and k // (2 * least) >= 64:
            least *= 2
        least = min(least, 56)
        per = -(-(-(-k // least)) // 16) * 16
        launch = probe.exact_grad(m, n, k)[0]
        assert launch.name == "exact"
        assert least == 1 or launch.splits >= -(-k // per), (m, n, k, least, launch.splits)


def fields(x):
    return (x.name, x.tile_m, x.tile_n, x.kgroups, x.splits, x.k_per_split, x.whole, x.split_tiles)


def test_own_plan_passed_in_launches_the_same():
    """A plan equal to the library's launches what the library launches: the
    same kernel, tiles and K slices."""
    rng = random.Random(6)
    sizes = [(976, 1264, 596, 1), (1738, 538, 3079, 1), (1438, 1285, 1100, 1), (256, 256, 256, 1), (70, 70, 1000, 1)]
    sizes += [(log_uniform(rng, 1, 5000), log_uniform(rng, 1, 5000), log_uniform(rng, 1, 20000), rng.choice([1, 1, 3, 50]))
              for _ in range(1500)]
    kinds = set()
    for m, n, k, batch in sizes:
        for workspace, limit in ((True, None), (False, 0)):
            own = probe.plan(m, n, k, batch, max_workspace_bytes=limit)
            auto = [fields(x) for x in probe.product(m, n, k, batch, tb=False, workspace=workspace)]
            if limit == 0 and own == probe.plan(m, n, k, batch):
                continue
            assert [fields(x) for x in probe.product(m, n, k, batch, tb=False, plan=own)] == auto, (m, n, k, batch, own)
            kinds.add((auto[0][0], own[3], own[2] > 1))
    assert {("tiled", 2, True), ("tiled", 4, True), ("tiled", 1, True), ("small", 4, False)} <= kinds


def test_callers_plan_runs_its_tiles():
    """A plan that is not the library's runs the tiled kernel as given."""
    for plan in ((64, 64, 1, 4, 1), (64, 64, 3, 4, 0), (128, 64, 1, 2, 1), (128, 128, 2, 1, 1)):
        for m, n, k in ((256, 128, 272), (70, 66, 300), (8, 64, 4096)):
            got = probe.product(m, n, k, plan=plan)
            assert (got[0].name, got[0].tile_m, got[0].tile_n, got[0].kgroups) == ("tiled", plan[0], plan[1], plan[3])


def parameters(function, names):
    return [case for mark in function.pytestmark if mark.name == "parametrize" and mark.args[0] == names
            for case in mark.args[1]]


def test_gpu_tests_reach_the_kernels_they_name():
    """The sizes of the GPU tests of each kernel do go to that kernel."""
    import test_gpu_bf16
    import test_gpu_skinny
    import test_gpu_small
    layouts = ((False, False), (False, True), (True, False), (True, True))
    sizes = parameters(test_gpu_small.test_sizes_and_layouts, "m,n,k")
    assert len(sizes) >= 9
    for m, n, k in sizes + [(70, 66, 300), (64, 64, 128), (45, 77, 203), (33, 40, 5)]:
        for ta, tb in layouts:
            assert names(probe.product(m, n, k, ta=ta, tb=tb)) == ["small"], (m, n, k, ta, tb)
    fews = parameters(test_gpu_skinny.test_row_counts_widths_and_k, "few")
    wides = parameters(test_gpu_skinny.test_row_counts_widths_and_k, "wide,k")
    assert len(fews) >= 10 and len(wides) >= 6
    for few in fews:
        for wide, k in wides:
            if min(few, wide) <= 32:
                for m, n in ((few, wide), (wide, few)):
                    assert names(probe.product(m, n, k)) == ["few rows"], (m, n, k)
    long_k = parameters(test_gpu_skinny.test_long_k_folds_its_sums, "few,wide,k")
    assert len(long_k) >= 4
    for few, wide, k in long_k:
        assert names(probe.product(few, wide, k, workspace=False)) == ["few rows"]
    for shape, kind in test_gpu_bf16.PLAN_SHAPES:
        for size in (shape, (*(-(-d // 8) * 8 for d in shape[:3]), shape[3])):
            for ta, tb in layouts:
                got = probe.product(*size, ta=ta, tb=tb, bf16=True)[0]
                assert (got.name, got.tile_m, got.tile_n, got.kgroups) == ("tiled", *kind[:3]), (size, ta, tb)
