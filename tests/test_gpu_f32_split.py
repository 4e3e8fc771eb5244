"""GPU parity of the three fp32 products: operands split into bf16 parts (tiles 64 and 128), the fp32 matrix
instruction (forced as 16) and the short product (32), each against the fp64 oracle or a wider sum.

Bound for normal inputs: see test_gpu_f32.py (TOL_F32)."""
import numpy as np
import pytest
import torch

from paper_2406_17660_amd import grass
from gpu_util import DEV, TOL_F32, rel_fro, to_f64, to_np
from test_gpu_f32 import _inputs, _want

pytestmark = pytest.mark.gpu
KERNELS = [16, 32, 64, 128]


@pytest.mark.parametrize("kernel", KERNELS)
@pytest.mark.parametrize("layout", [grass.DY_TxM, grass.DY_MxT])
@pytest.mark.parametrize("T,m,n,r", [
    (1, 3, 2, 2), (31, 40, 33, 32), (33, 64, 31, 33), (257, 70, 65, 5), (511, 90, 97, 65), (1055, 130, 129, 40)])
def test_every_kernel_at_edges(kernel, layout, T, m, n, r):
    """Ragged tokens, rows and columns, odd numbers of K tiles (one half of a slice then has a turn less),
    with as many slices as the workspace allows and with one."""
    dY, X, idx, rho = _inputs(T, m, n, r, layout, seed=T)
    want = _want(dY, X, idx, rho, layout)
    grass.set_test_option(grass.TEST_GEMM_TILE, kernel)
    for cap in (0, 1, 3):
        grass.set_test_option(grass.TEST_MAX_K_SLICES, cap)
        GC = torch.full((r, n), float("nan"), device=DEV)
        need = grass.cgrad_workspace(T, m, n, r, grass.F32, layout)
        grass.compressed_grad(dY, X, idx, rho, GC, grass.workspace(need) if need else None, layout)
        assert rel_fro(to_np(GC), want) <= TOL_F32


@pytest.mark.parametrize("kernel", KERNELS)
@pytest.mark.parametrize("low,high", [(-149, -130), (-140, -100), (-102, -98), (-130, 20), (100, 127)])
def test_magnitudes_that_bf16_parts_do_not_hold(kernel, low, high):
    """Values between 2^low and 2^high.  A sum of T products is off by at most T * 2^-24 of the sum of
    their magnitudes, and by half a subnormal step per addition."""
    T, m, n = 200, 40, 36
    g = torch.Generator(device=DEV)
    g.manual_seed(1)
    e = torch.rand((T, m), generator=g, device=DEV, dtype=torch.float64) * (high - low) + low
    sign = torch.randint(0, 2, (T, m), generator=g, device=DEV) * 2 - 1
    dY = (sign * 2.0 ** e).float()
    X = (torch.randn((T, n), generator=g, device=DEV) * 2.0 ** (10 - (high if high > 0 else low) / 2)).float()
    grass.set_test_option(grass.TEST_GEMM_TILE, kernel)
    G = torch.full((m, n), float("nan"), device=DEV)
    grass.dense_grad(dY, X, G, grass.workspace(max(16, grass.dense_workspace(T, m, n, grass.F32))))
    want = dY.double().t() @ X.double()
    bound = T * 2.0 ** -24 * (dY.double().abs().t() @ X.double().abs()) + T * 2.0 ** -149
    assert bool(((G.double() - want).abs() <= bound).all())


@pytest.mark.parametrize("kernel", KERNELS)
@pytest.mark.parametrize("low,high", [(-75, -50), (-149, -60), (40, 44), (52, 56)])
def test_small_and_large_products(kernel, low, high):
    """Both operands between 2^low and 2^high: products below the smallest normal value, and sums around 2^80.
    The bound of the test above."""
    T, m, n = 200, 40, 36
    g = torch.Generator(device=DEV)
    g.manual_seed(3)
    dY, X = (((torch.randint(0, 2, (T, w), generator=g, device=DEV) * 2 - 1) * 2.0 ** (
        torch.rand((T, w), generator=g, device=DEV, dtype=torch.float64) * (high - low) + low)).float() for w in (m, n))
    grass.set_test_option(grass.TEST_GEMM_TILE, kernel)
    G = torch.full((m, n), float("nan"), device=DEV)
    grass.dense_grad(dY, X, G, grass.workspace(grass.dense_workspace(T, m, n, grass.F32)))
    want = dY.double().t() @ X.double()
    bound = T * 2.0 ** -24 * (dY.double().abs().t() @ X.double().abs()) + T * 2.0 ** -149
    assert bool(((G.double() - want).abs() <= bound).all())


@pytest.mark.parametrize("kernel", KERNELS)
@pytest.mark.parametrize("T", [40, 1100])
def test_tiny_values_leave_other_outputs_as_they_are(kernel, T):
    """The bits of an output depend on its own column and row alone: values of 2^-110 and subnormal ones elsewhere
    in the tile are multiplied like all others, and cost nothing more."""
    m, n = 140, 136
    g = torch.Generator(device=DEV)
    g.manual_seed(4)
    dY, X = torch.randn((T, m), generator=g, device=DEV), torch.randn((T, n), generator=g, device=DEV)
    grass.set_test_option(grass.TEST_GEMM_TILE, kernel)
    ws = grass.workspace(grass.dense_workspace(T, m, n, grass.F32))
    G, H = (torch.full((m, n), float("nan"), device=DEV) for _ in range(2))
    grass.dense_grad(dY, X, G, ws)
    dY[T // 2, 3], dY[T - 1, 70], X[0, 100] = 2.0 ** -110, 2.0 ** -149, -2.0 ** -127
    grass.dense_grad(dY, X, H, ws)
    assert bool(torch.isfinite(H).all())
    same = torch.ones((m, n), dtype=torch.bool, device=DEV)
    same[[3, 70]], same[:, 100] = False, False
    assert torch.equal(G[same], H[same])


@pytest.mark.parametrize("kernel", KERNELS)
def test_infinities_and_nan_stay_where_they_belong(kernel):
    """An output is not finite exactly where the product of its own column and row is not; the largest
    finite values (which round to an infinite bf16) stay finite."""
    T, m, n = 70, 40, 37
    g = torch.Generator(device=DEV)
    g.manual_seed(2)
    dY, X = torch.rand((T, m), generator=g, device=DEV) + 0.5, torch.rand((T, n), generator=g, device=DEV) * 1e-3 + 1e-3
    big = torch.finfo(torch.float32).max
    dY[3, 1], dY[69, 2], dY[5, 3], dY[7, 4], dY[:, 5] = float("inf"), -float("inf"), float("nan"), big, 0.0
    X[4, 6], X[3, 7] = float("inf"), 0.0
    grass.set_test_option(grass.TEST_GEMM_TILE, kernel)
    G = torch.empty((m, n), device=DEV)
    grass.dense_grad(dY, X, G, grass.workspace(max(16, grass.dense_workspace(T, m, n, grass.F32))))
    want = (dY.double().cpu().t() @ X.double().cpu()).numpy()
    got = to_f64(G)
    assert np.array_equal(np.isnan(got), np.isnan(want)) and np.array_equal(np.isinf(got), np.isinf(want))
    fine = np.isfinite(want)
    assert np.array_equal(got[np.isinf(want)], want[np.isinf(want)])
    assert np.abs(got[fine] / np.where(want[fine] == 0, 1, want[fine]) - (want[fine] != 0)).max() <= T * 2.0 ** -24


@pytest.mark.parametrize("sdt", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("wdt", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("T,n,rs,layout", [(512, 256, (16,), grass.DY_TxM), (100, 33, (32, 1, 7), grass.DY_TxM),
                                           (17, 40, (31, 32), grass.DY_MxT)])
def test_step_in_one_launch_equals_the_one_in_two(sdt, wdt, T, n, rs, layout):
    """Adam and the row update inside the short product (runs of repeated rows, groups, G_C stored or not)
    against the same step with events on its kernels, which runs them as two: bit for bit."""
    m = 20
    X = torch.randn(T, n, device=DEV)
    sets = []
    for k, r in enumerate(rs):
        dY, _, idx, rho = _inputs(T, m, n, r, layout, seed=k)
        sets.append((dY, idx, rho, torch.randn(r, n, device=DEV).to(sdt), torch.rand(r, n, device=DEV).to(sdt),
                     torch.randn(m, n, device=DEV).to(wdt)))
    ws = grass.workspace(grass.step_group_workspace(T, n, rs, grass.F32, layout))
    events = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    for e in events:
        e.record()
    results = []
    for gemm_events in (None, events):
        dYs, idxs, rhos, Ms, Vs, Ws = (list(t) for t in zip(*[(s[0], s[1], s[2], *(x.clone() for x in s[3:])) for s in sets]))
        GCs = [torch.full((r, n), float("nan"), device=DEV) if k != 1 else None for k, r in enumerate(rs)]
        grass.step_group(dYs, X, idxs, rhos, Ms, Vs, Ws, 1e-2, 0.9, 0.999, 1e-8, 3, 0.5, ws, layout, GCs=GCs,
                         gemm_events=gemm_events)
        results.append([*Ms, *Vs, *Ws, *(G for G in GCs if G is not None)])
    for a, b in zip(*results):
        assert torch.equal(a, b)


@pytest.mark.parametrize("T", [1, 2, 3, 5, 7])
def test_few_tokens_take_exact_products(T):
    """Below 8 tokens the products are those of the fp32 instruction, whatever the shape, in separate calls and in
    steps: one token gives the correctly rounded product of the two values."""
    g = torch.Generator(device=DEV)
    g.manual_seed(T)
    for m, n, r in ((40, 96, 32), (6400, 6400, 6400)):  # a single row tile; more than 0.3 Gflop from T = 4 on
        # mantissas whose parts are as large as they get, and random ones
        dY = torch.where(torch.rand((T, m), generator=g, device=DEV) < 0.5, float.fromhex("0x1.00ff8p+0"), 0.0)
        dY += torch.randn((T, m), generator=g, device=DEV) * (dY == 0)
        X = torch.where(torch.rand((T, n), generator=g, device=DEV) < 0.5, float.fromhex("0x1.00ff8p+0"), 0.0)
        X += torch.randn((T, n), generator=g, device=DEV) * (X == 0)
        idx, rho = torch.arange(r, dtype=torch.int32, device=DEV), torch.ones(r, device=DEV)
        results = []
        for kernel in (0, 16):
            grass.set_test_option(grass.TEST_GEMM_TILE, kernel)
            GC, G = (torch.full((r, n), float("nan"), device=DEV) for _ in range(2))
            grass.compressed_grad(dY, X, idx, rho, GC, None)
            M, V, W = (torch.zeros(s, n, device=DEV) for s in (r, r, m))
            grass.step_group([dY], X, [idx], [rho], [M], [V], [W], 1e-2, 0.9, 0.999, 1e-8, 1, 0.5,
                             grass.workspace(grass.step_group_workspace(T, n, [r], grass.F32)), GCs=[G])
            results.append((GC, G))
        for a, b in zip(*results):
            assert torch.equal(a, b)
        if T == 1:
            assert torch.equal(results[0][0], dY.t()[:r] * X)


def _spread(t, ld):
    """`t` with rows ld elements apart, the gaps left as they are."""
    buf = torch.empty((t.shape[0] - 1) * ld + t.shape[1], device=DEV)
    view = buf.as_strided(t.shape, (ld, 1))
    view.copy_(t)
    return view


def _products_and_step(dY, X, idx, rho, layout, kernel):
    (T, n), r = X.shape, idx.shape[0]
    m = dY.shape[1] if layout == grass.DY_TxM else dY.shape[0]
    grass.set_test_option(grass.TEST_GEMM_TILE, kernel)
    ws = grass.workspace(max(grass.step_group_workspace(T, n, [r], grass.F32, layout),
                             grass.dense_workspace(T, m, n, grass.F32, layout)))
    GC, G, M, V, W = (torch.zeros(k, n, device=DEV) for k in (r, m, r, r, m))
    grass.compressed_grad(dY, X, idx, rho, GC, ws, layout)
    grass.dense_grad(dY, X, G, ws, layout)
    grass.step_group([dY], X, [idx], [rho], [M], [V], [W], 1e-2, 0.9, 0.999, 1e-8, 1, 0.5, ws, layout)
    return GC, G, M, V, W


@pytest.mark.parametrize("kernel", [32, 64, 128])
@pytest.mark.parametrize("T,ld,m", [(50, 1 << 24, 63), (50, 1 << 24, 64), (43, (1 << 24) + 3, 90), (70, 1 << 27, 10)])
def test_rows_of_mxt_storage_may_lie_anywhere(kernel, T, ld, m):
    """A dY stored m x T whose rows reach past 2^30 elements (and one just below): the same kernel, the same bits as
    with rows next to each other."""
    n, r = 70, min(m, 40)
    dY, X, _, rho = _inputs(T, m, n, r, grass.DY_MxT, seed=ld % 97)
    idx = torch.arange(m - r, m, dtype=torch.int32, device=DEV)
    want = _products_and_step(dY, X, idx, rho, grass.DY_MxT, kernel)
    assert rel_fro(to_np(want[0]), _want(dY, X, idx, rho, grass.DY_MxT)) <= TOL_F32
    for a, b in zip(_products_and_step(_spread(dY, ld), X, idx, rho, grass.DY_MxT, kernel), want):
        assert torch.equal(a, b)


@pytest.mark.parametrize("kernel", [0, 32, 64, 128])
@pytest.mark.parametrize("ldy,ldx", [((1 << 24) - 1, 64), (48, (1 << 24) - 1), (1 << 24, 64), (48, (1 << 24) + 1)])
def test_row_strides_around_32_bit_offsets(kernel, ldy, ldx):
    """From row strides of 2^24 on the kernel that addresses in 64 bits runs, whatever the size; below, the chosen
    one.  Same bits as with rows next to each other."""
    T, m, n, r = 41, 48, 64, 30
    dY, X, idx, rho = _inputs(T, m, n, r, grass.DY_TxM, seed=7)
    want = _products_and_step(dY, X, idx, rho, grass.DY_TxM, 16 if max(ldy, ldx) >= 1 << 24 else kernel)
    got = _products_and_step(_spread(dY, ldy) if ldy > m else dY, _spread(X, ldx) if ldx > n else X, idx, rho,
                             grass.DY_TxM, kernel)
    for a, b in zip(got, want):
        assert torch.equal(a, b)


@pytest.mark.parametrize("kernel,T,m,n,rs,layout", [
    (32, 512, 256, 256, (16,), grass.DY_TxM),       # one round of short workgroups
    (32, 500, 3000, 2048, (32,), grass.DY_MxT),     # nothing to gather
    (32, 300, 128, 5000, (20, 3), grass.DY_TxM),    # two rounds, 64 tokens and more
    (16, 63, 128, 5000, (20, 3), grass.DY_TxM),     # two rounds, fewer
    (16, 512, 256, 5500, (32, 32, 32), grass.DY_TxM),  # more than two
    (16, 503, 603, 64, (31, 31), grass.DY_TxM),     # more gathered lines than a short workgroup fetches in time
    (16, 1344, 512, 352, (37,), grass.DY_TxM),      # below 0.3 Gflop
    (128, 98, 2904, 9776, (55, 55, 55), grass.DY_TxM),  # the gather bounds it: fewest column tiles
    (128, 1344, 5905, 6339, (37,), grass.DY_TxM),
    (128, 8192, 1024, 1024, (256,), grass.DY_TxM),
    (64, 1024, 1024, 4096, (40,), grass.DY_MxT),
])
def test_the_kernel_a_step_runs_with(kernel, T, m, n, rs, layout):
    """Which kernel is chosen, told by the bits of the results: those of the one that is forced, and of no other."""
    X, sets = torch.randn(T, n, device=DEV), []
    for k, r in enumerate(rs):
        dY, _, idx, rho = _inputs(T, m, n, r, layout, seed=k)
        sets.append((dY, idx, rho))
    results = {}
    for forced in (0, *KERNELS):
        if forced == 32 and max(rs) > 32:
            continue
        grass.set_test_option(grass.TEST_GEMM_TILE, forced)
        Ms, Vs, GCs = ([torch.zeros(r, n, device=DEV) for r in rs] for _ in range(3))
        Ws = [torch.zeros(m, n, device=DEV) for _ in rs]
        dYs, idxs, rhos = (list(t) for t in zip(*sets))
        grass.step_group(dYs, X, idxs, rhos, Ms, Vs, Ws, 1e-2, 0.9, 0.999, 1e-8, 1, 0.5,
                         grass.workspace(grass.step_group_workspace(T, n, rs, grass.F32, layout)), layout, GCs=GCs)
        results[forced] = torch.cat(GCs)
    assert [k for k in KERNELS if k in results and torch.equal(results[k], results[0])] == [kernel]
