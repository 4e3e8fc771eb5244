"""What the workspace queries promise, from the library's host functions alone: the partial tiles a
planned product writes fit into the workspace its query asks for."""
import numpy as np
import pytest

from paper_2406_17660_amd import grass


def narrow_partial_bytes(T, n, rs, m):
    """Bytes of partial tiles of the kernel that gathers by itself (the tiles are 256 columns wide and
    the rows of all sets lie in one panel, each set rounded up to 8 rows), or None where another
    kernel is planned."""
    panel = sum((r + 7) // 8 * 8 for r in rs)
    tile, slices = grass.cgrad_plan(T, n, panel if len(rs) > 1 else rs[0], grass.BF16, m=m, count=len(rs))
    return slices * panel * ((n + 255) // 256 * 256) * 4 if tile == 0 else None


def narrow_workspace(T, n, rs, m):
    return (grass.cgrad_workspace(T, m, n, rs[0], grass.BF16) if len(rs) == 1
            else grass.cgrad_group_workspace(T, n, rs, grass.BF16))


@pytest.mark.parametrize("sets", range(1, 9))
def test_partial_tiles_of_narrow_groups_fit_the_queried_workspace(sets):
    """One to eight sets, equal and unequal ranks, over the kernel's whole range.  255 bytes of the
    workspace may go into aligning its start."""
    rng = np.random.default_rng(sets)
    narrow = 0
    for k in range(400):
        T = int(2 ** rng.uniform(4, 17)) // 16 * 16
        n, m = int(rng.integers(1, 65)) * 8, int(rng.integers(1, 65)) * 8
        rs = [int(rng.integers(1, 129))] * sets if k % 2 else [int(r) for r in rng.integers(1, 129, sets)]
        used = narrow_partial_bytes(T, n, rs, m)
        if used is None:
            continue
        narrow += 1
        assert used + 255 <= narrow_workspace(T, n, rs, m), (T, n, m, rs)
        step = grass.step_group_workspace(T, n, rs, grass.BF16)
        # a step keeps an unnamed G_C of each set behind the partial tiles
        assert used + 255 + sum(r * n * 4 for r in rs) <= step, (T, n, m, rs)
    assert narrow > 300


@pytest.mark.parametrize("T,n,m,rs", [(8192, 512, 512, [32] * 8), (2048, 256, 512, [32] * 8),
                                      (480, 256, 512, [64] * 4), (1024, 64, 512, [32] * 8)])
def test_narrow_groups_of_many_slices_fit(T, n, m, rs):
    """Groups whose slice count is bounded by the room for the partial tiles."""
    used = narrow_partial_bytes(T, n, rs, m)
    assert used is not None and used + 255 <= narrow_workspace(T, n, rs, m)


@pytest.mark.parametrize("layout", [grass.DY_TxM, grass.DY_MxT])
@pytest.mark.parametrize("T,n,r", [(1, 64, 16), (512, 256, 16), (1023, 300, 200), (1024, 4096, 4096), (2048, 11008, 4096),
                                   (4096, 4096, 4096), (8192, 2048, 2048), (8192, 1024, 256), (8192, 64, 33)])
def test_fp32_products_of_one_slice_ask_for_no_workspace(T, n, r, layout):
    """Partial tiles are written for several slices, or for the tail of a step; the sums of one slice go to the
    output."""
    _, slices = grass.cgrad_plan(T, n, r, grass.F32, layout)
    sizes = [grass.cgrad_workspace(T, r, n, r, grass.F32, layout), grass.dense_workspace(T, r, n, grass.F32, layout)]
    assert all((size == 0) == (slices == 1) for size in sizes), (slices, sizes)


# Ragged token counts: bytes that the queries once asked for, with the tokens past the last whole K tile as a slice of
# their own.  A program that keeps the size of its workspace is still served.
@pytest.mark.parametrize("call,T,rows,n,layout,size", [
    (grass.CALL_CGRAD, 496, 8, 72, grass.DY_TxM, 778496), (grass.CALL_CGRAD, 4338, 8, 128, grass.DY_TxM, 6415616),
    (grass.CALL_CGRAD, 4578, 16, 160, grass.DY_MxT, 6800640), (grass.CALL_CGRAD, 4600, 4, 3, grass.DY_TxM, 6885632),
    (grass.CALL_DENSE, 5105, 11, 61, grass.DY_MxT, 8248320), (grass.CALL_DENSE, 5358, 8, 160, grass.DY_TxM, 5243136),
    (grass.CALL_CGRAD, 6378, 48, 180, grass.DY_TxM, 11904512), (grass.CALL_CGRAD, 6884, 115, 11, grass.DY_MxT, 10298880),
    (grass.CALL_DENSE, 6910, 71, 10, grass.DY_TxM, 10312960),
    (grass.CALL_STEP, 496, 8, 72, grass.DY_TxM, 778496 + 256 + 8 * 72 * 4)])
def test_sizes_once_asked_for_are_accepted(call, T, rows, n, layout, size):
    assert grass.least_workspace(call, T, n, [rows], layout) <= size


@pytest.mark.parametrize("layout", [grass.DY_TxM, grass.DY_MxT])
def test_the_least_workspace_is_part_of_the_query(layout):
    rng = np.random.default_rng(3)
    for _ in range(300):
        T, n = int(2 ** rng.uniform(0, 16)), int(2 ** rng.uniform(0, 12))
        rs = [int(2 ** rng.uniform(0, 10)) for _ in range(rng.integers(1, 5))]
        assert grass.least_workspace(grass.CALL_CGRAD, T, n, rs[:1], layout) <= grass.cgrad_workspace(T, rs[0], n, rs[0], grass.BF16, layout)
        assert grass.least_workspace(grass.CALL_DENSE, T, n, rs[:1], layout) <= grass.dense_workspace(T, rs[0], n, grass.BF16, layout)
        assert grass.least_workspace(grass.CALL_STEP, T, n, rs, layout) <= grass.step_group_workspace(T, n, rs, grass.BF16, layout)


@pytest.mark.parametrize("T,n,rows,layout", [(5018, 8288, 785, grass.DY_MxT), (5647, 9336, 889, grass.DY_TxM),
                                             (7833, 2072, 334, grass.DY_TxM), (6637, 2745, 3371, grass.DY_TxM)])
def test_slices_are_not_longer_than_those_planned_by_themselves(T, n, rows, layout):
    rng = np.random.default_rng(T)
    shapes = [(T, n, rows)] + [(int(2 ** rng.uniform(5, 13)), int(2 ** rng.uniform(3, 13.4)), int(2 ** rng.uniform(3, 12)))
                               for _ in range(2000)]
    found = [grass.cgrad_plan(T, n, rows, grass.BF16, layout)[1] for T, n, rows in shapes]
    grass.set_test_option(grass.TEST_MAX_K_SLICES, 128)  # the slices planned by themselves
    alone = [grass.cgrad_plan(T, n, rows, grass.BF16, layout)[1] for T, n, rows in shapes]
    assert [s for s, f, a in zip(shapes, found, alone) if f < a] == []


@pytest.mark.parametrize("T,n,m,r,count", [(21936, 448, 248, 3, 3), (12960, 16, 488, 41, 8), (31392, 416, 160, 1, 3),
                                           (19792, 8, 504, 38, 4), (16368, 368, 440, 1, 3), (12320, 24, 480, 36, 8)])
def test_slices_of_narrow_layers_are_not_longer_than_by_the_traffic_rule(T, n, m, r, count):
    """Two workgroups per compute unit, a quarter of the inputs' bytes, four K tiles of 16 tokens at least, 128 slices."""
    tile, slices = grass.cgrad_plan(T, n, (r + 7) // 8 * 8 * count, grass.BF16, m=m, count=count)
    ktiles, tiles, slice_bytes = T // 16, count * ((n + 255) // 256), (r + 7) // 8 * 8 * count * ((n + 255) // 256) * 1024
    rule = max(1, min(-(-512 // tiles), T * (m * count + n) // 2 // slice_bytes, ktiles // 4, 128))
    assert tile == 0 and -(-ktiles // slices) <= -(-ktiles // rule)


@pytest.mark.parametrize("T,n,rows", [(5365, 608, 1472), (271, 416, 512), (137, 216, 512), (2119, 256, 208)])
def test_plan_names_the_tile_whose_slices_it_names(T, n, rows):
    """Planned by themselves these slices are the large tile's; the quicker ones are a smaller tile's own."""
    grass.set_test_option(grass.TEST_MAX_K_SLICES, 128)
    alone = grass.cgrad_plan(T, n, rows, grass.BF16)
    grass.set_test_option(grass.TEST_MAX_K_SLICES, 0)
    tile, slices = grass.cgrad_plan(T, n, rows, grass.BF16)
    assert alone[0] == 256 and slices > alone[1] and tile == 128


@pytest.mark.parametrize("T,n,rows", [(1600, 136, 1232), (6848, 5048, 448), (4928, 392, 312), (704, 512, 760)])
def test_plan_of_a_group_stored_mxt_packs(T, n, rows):
    """The rows of several sets are packed; only those of a single one are gathered by the product itself."""
    group = grass.cgrad_plan(T, n, rows, grass.BF16, grass.DY_MxT, count=2)
    grass.set_test_option(grass.TEST_PACK_MXT, 1)
    assert grass.cgrad_plan(T, n, rows, grass.BF16, grass.DY_MxT, count=2) == group


@pytest.mark.parametrize("tile,direct", [(128, 1), (128, 0), (192, 1), (256, 1), (256, 0)])
def test_estimate_does_not_fall_when_work_is_added(tile, direct):
    f = grass.lib().grass_test_product_us
    for ktiles in (1, 2, 4, 8, 10, 11, 16, 32, 100, 1000):
        times = [f(tile, direct, wgs, ktiles) for wgs in range(1, 2600)]
        assert times == sorted(times), (ktiles, [w for w in range(1, 2599) if times[w] < times[w - 1]][:4])
    for wgs in (1, 100, 256, 257, 512, 768, 769, 3000):
        times = [f(tile, direct, wgs, k) for k in range(1, 300)]
        assert times == sorted(times)
