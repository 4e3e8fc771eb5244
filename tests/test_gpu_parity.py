"""GPU parity: every C-ABI entry point against the fp64 CPU oracle on the same seeded inputs.

Bars: selected indices bit-exact; floating-point results within a relative Frobenius error
of 1e-5 (fp32 inputs) / 1e-2 (bf16 inputs), with tighter elementwise checks where the
arithmetic allows them.
"""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_2406_17660_amd import grass, workloads
from gpu_util import (DEV, TOL_BF16, TOL_F32, bf16_ulp, gpu_cgrad, gpu_dense, gpu_select, rel_fro,
                      to_f64, to_np, tol_for)

pytestmark = pytest.mark.gpu

LR, B1, B2, EPS = 1e-3, 0.9, 0.999, 1e-8


def randn(shape, dtype, seed, scale=1.0, ld=None):
    """Seeded N(0, scale^2) device tensor; with ld > cols it is a view into a wider buffer."""
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    rows, cols = shape
    ld = cols if ld is None else ld
    buf = (torch.randn((rows, ld), generator=g, device=DEV) * scale).to(dtype)
    return buf[:, :cols] if ld != cols else buf


# ------------------------------------------------------------------------------ row stats
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("m,n,ld", [(1, 1, 1), (5, 7, 7), (256, 256, 256), (300, 1000, 1024),
                                    (64, 333, 333), (1376, 512, 512), (33, 4099, 4104),
                                    (7, 0, 4), (3, 5461, 5461)])
def test_row_stats(dtype, m, n, ld):
    G = randn((m, n), dtype, 100 + m + n, ld=ld)
    out = torch.full((m,), float("nan"), dtype=torch.float32, device=DEV)
    grass.row_stats(G, out)
    want = ref.row_stats(to_np(G)) if n > 0 else np.zeros(m)
    got = to_f64(out)
    assert rel_fro(got, want) <= TOL_F32  # fp32 accumulation of exactly widened inputs
    np.testing.assert_allclose(got, want, rtol=2e-6, atol=0)


def test_row_stats_empty():
    G = torch.zeros((0, 8), device=DEV)
    out = torch.zeros((0,), device=DEV)
    grass.row_stats(G, out)


# ------------------------------------------------------------------------------ selection
METHODS = [(grass.SEL_TOPR, False), (grass.SEL_UNIFORM, True), (grass.SEL_UNIFORM, False),
           (grass.SEL_MULTI_NORM, True), (grass.SEL_MULTI_NORM, False),
           (grass.SEL_MULTI_NORM2, True), (grass.SEL_MULTI_NORM2, False)]


def sumsq_case(m, kind, seed):
    rng = np.random.default_rng(seed)
    if kind == "chi2":
        s = rng.standard_normal(m) ** 2 * 100
    elif kind == "lognormal":
        s = np.exp(2 * rng.standard_normal(m))
    elif kind == "ties":
        s = rng.integers(0, 4, m).astype(np.float64)  # many equal values and zeros
    elif kind == "zeros":
        s = np.zeros(m)
    elif kind == "tiny":
        s = rng.standard_normal(m) ** 2 * 1e-40  # denormals
    elif kind == "wide":
        s = 10.0 ** rng.uniform(-30, 30, m)  # sixty decades: most quantised weights are 1
    elif kind == "one_hot":
        s = np.zeros(m)
        s[m // 3] = 7.0  # a single row carries all the weight
    elif kind == "equal":
        s = np.full(m, 3.25)
    else:
        raise ValueError(kind)
    return s.astype(np.float32)


@pytest.mark.parametrize("method,replacement", METHODS)
@pytest.mark.parametrize("m,r,kind", [(1, 1, "chi2"), (5, 3, "chi2"), (64, 64, "lognormal"),
                                      (65, 17, "ties"), (1000, 128, "chi2"), (1000, 999, "ties"),
                                      (4097, 1024, "lognormal"), (512, 128, "zeros"),
                                      (300, 100, "tiny"), (13824, 1024, "chi2"),
                                      (2000, 300, "wide"), (777, 50, "one_hot"), (640, 640, "equal")])
def test_select_rows_bit_exact(method, replacement, m, r, kind):
    ss = sumsq_case(m, kind, 7 * m + r)
    d_ss = torch.from_numpy(ss).to(DEV)
    for seed, refresh in [(0, 0), (0x9E3779B97F4A7C15, 12345678901)]:
        idx, rho, status = gpu_select(d_ss, r, method, replacement, seed=seed, refresh_id=refresh)
        assert status == grass.OK
        w_idx, w_rho, _ = ref.select_rows(ss, r, method, replacement, seed=seed, refresh_id=refresh)
        assert np.array_equal(idx.cpu().numpy(), w_idx), (method, replacement, m, r, kind)
        assert np.array_equal(rho.cpu().numpy(), w_rho)  # same IEEE double ops, one rounding
        if method == grass.SEL_TOPR:
            break


@pytest.mark.parametrize("method", [grass.SEL_UNIFORM, grass.SEL_MULTI_NORM])
@pytest.mark.parametrize("scale", [grass.SCALE_ONE, grass.SCALE_INV_SQRT_RQ])
def test_select_forced_scale(method, scale):
    ss = sumsq_case(777, "lognormal", 3)
    d_ss = torch.from_numpy(ss).to(DEV)
    for replacement in (True, False):
        idx, rho, status = gpu_select(d_ss, 200, method, replacement, scale, seed=11, refresh_id=2)
        w_idx, w_rho, _ = ref.select_rows(ss, 200, method, replacement, scale, seed=11, refresh_id=2)
        assert status == grass.OK
        assert np.array_equal(idx.cpu().numpy(), w_idx)
        assert np.array_equal(rho.cpu().numpy(), w_rho)


def test_select_more_draws_than_rows_with_replacement():
    ss = sumsq_case(10, "chi2", 5)
    idx, rho, status = gpu_select(torch.from_numpy(ss).to(DEV), 50, grass.SEL_MULTI_NORM, True, seed=4)
    w_idx, w_rho, _ = ref.select_rows(ss, 50, grass.SEL_MULTI_NORM, True, seed=4)
    assert status == grass.OK and np.array_equal(idx.cpu().numpy(), w_idx)
    assert np.array_equal(rho.cpu().numpy(), w_rho)


@pytest.mark.parametrize("m,r", [(20000, 1500), (300001, 2000)])
def test_select_without_replacement_tree_in_global_memory(m, r):
    """m too large for the LDS-resident sum tree: 3 and 4 level trees in the workspace."""
    ss = sumsq_case(m, "lognormal", m)
    idx, rho, status = gpu_select(torch.from_numpy(ss).to(DEV), r, grass.SEL_MULTI_NORM, False, seed=9)
    w_idx, _, _ = ref.select_rows(ss, r, grass.SEL_MULTI_NORM, False, seed=9)
    assert status == grass.OK and np.array_equal(idx.cpu().numpy(), w_idx)


@pytest.mark.parametrize("bad", [float("nan"), float("inf"), -1.0])
@pytest.mark.parametrize("method,replacement", [(grass.SEL_TOPR, False), (grass.SEL_MULTI_NORM, True),
                                                (grass.SEL_MULTI_NORM, False)])
def test_select_reports_nonfinite(bad, method, replacement):
    ss = sumsq_case(100, "chi2", 1)
    ss[37] = bad
    idx, rho, status = gpu_select(torch.from_numpy(ss).to(DEV), 10, method, replacement)
    assert status == grass.ERR_NONFINITE
    with pytest.raises(ref.OracleError) as e:
        ref.select_rows(ss, 10, method, replacement)
    assert e.value.code == ref.ERR_NONFINITE
    i = idx.cpu().numpy()
    assert i.min() >= 0 and i.max() < 100 and (np.diff(i) >= 0).all()  # placeholder stays in bounds
    assert (rho.cpu().numpy() == 1.0).all()


def test_select_zero_rows():
    ss = torch.ones(16, device=DEV)
    idx, rho, status = gpu_select(ss, 0, grass.SEL_TOPR, False)
    assert status == grass.OK and idx.numel() == 0


# ------------------------------------------------------------------------------ products
def make_idx(m, r, seed, duplicates):
    rng = np.random.default_rng(seed)
    if duplicates:
        idx = np.sort(rng.integers(0, m, r))
    else:
        idx = np.sort(rng.choice(m, r, replace=False))
    rho = rng.uniform(0.5, 2.0, r).astype(np.float32)
    return idx.astype(np.int32), rho


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("layout", [grass.DY_TxM, grass.DY_MxT])
@pytest.mark.parametrize("T,m,n,r,dup,pad", [
    (512, 256, 256, 16, False, 0),      # the fp32 reference configuration's shape
    (300, 200, 150, 37, True, 0),       # nothing divides a tile, duplicate rows
    (1000, 512, 1376, 128, False, 8),   # LLaMA-60M down-projection shape, padded leading dims
    (777, 130, 333, 129, True, 0),      # odd n: rows of X are not 16-byte aligned
    (64, 40, 24, 40, False, 0),         # r = m
    (4096, 300, 520, 260, False, 0),    # several K tiles per split, several tiles in both dims
])
def test_compressed_grad(dtype, layout, T, m, n, r, dup, pad):
    dY = randn((T, m), dtype, 1, scale=0.1, ld=m + pad)
    X = randn((T, n), dtype, 2, ld=n + pad)
    idx, rho = make_idx(m, r, 3, dup)
    d_idx, d_rho = torch.from_numpy(idx).to(DEV), torch.from_numpy(rho).to(DEV)
    dY_dev = dY if layout == grass.DY_TxM else dY.t().contiguous()
    GC = gpu_cgrad(dY_dev, X, d_idx, d_rho, layout)
    want = ref.compressed_grad(to_np(dY), to_np(X), idx, rho)
    got = to_f64(GC)
    assert np.isfinite(got).all()
    assert rel_fro(got, want) <= tol_for(dtype)
    # fp32 accumulation of exact products: far tighter than the bf16 contract
    assert rel_fro(got, want) <= 2e-5
    scale = np.abs(want).max()
    assert np.abs(got - want).max() <= 1e-4 * scale


def test_compressed_grad_empty_token_batch_and_empty_selection():
    X = torch.zeros((0, 64), dtype=torch.bfloat16, device=DEV)
    dY = torch.zeros((0, 32), dtype=torch.bfloat16, device=DEV)
    idx = torch.tensor([1, 5], dtype=torch.int32, device=DEV)
    rho = torch.ones(2, device=DEV)
    assert (gpu_cgrad(dY, X, idx, rho) == 0).all()
    X = randn((128, 64), torch.bfloat16, 1)
    dY = randn((128, 32), torch.bfloat16, 2)
    e = gpu_cgrad(dY, X, idx[:0], rho[:0])
    assert e.shape == (0, 64)


@pytest.mark.parametrize("dtype,gdtype", [(torch.float32, torch.float32),
                                          (torch.bfloat16, torch.float32),
                                          (torch.bfloat16, torch.bfloat16)])
@pytest.mark.parametrize("layout", [grass.DY_TxM, grass.DY_MxT])
@pytest.mark.parametrize("T,m,n", [(512, 256, 256), (300, 130, 150), (2048, 520, 264)])
def test_dense_grad_and_gather(dtype, gdtype, layout, T, m, n):
    dY = randn((T, m), dtype, 5, scale=0.1)
    X = randn((T, n), dtype, 6)
    dY_dev = dY if layout == grass.DY_TxM else dY.t().contiguous()
    G = gpu_dense(dY_dev, X, gdtype, layout)
    want = ref.full_grad(to_np(dY), to_np(X))
    assert rel_fro(to_f64(G), want) <= (TOL_BF16 if gdtype == torch.bfloat16 else 2e-5)
    # the naive comparator's second half: gather and scale selected rows (of a seeded matrix)
    Gs = randn((m, n), gdtype, 7)
    idx, rho = make_idx(m, min(m, 33), 8, True)
    out = torch.empty((len(idx), n), dtype=torch.float32, device=DEV)
    grass.gather_rows(Gs, torch.from_numpy(idx).to(DEV), torch.from_numpy(rho).to(DEV), out)
    want_rows = to_f64(Gs)[idx] * rho[:, None].astype(np.float64)
    np.testing.assert_allclose(to_f64(out), want_rows, rtol=1e-6, atol=0)


# ------------------------------------------------------------------------------ Adam / scatter
def adam_inputs(r, n, seed, ldgc):
    GC = randn((r, n), torch.float32, seed, scale=3.0, ld=ldgc)
    M = randn((r, n), torch.float32, seed + 1, scale=0.5)
    V = randn((r, n), torch.float32, seed + 2).square_()
    return GC, M.contiguous(), V.contiguous()


@pytest.mark.parametrize("r,n,ldgc", [(1, 1, 1), (16, 256, 256), (37, 1376, 1376), (5, 333, 333),
                                      (130, 1030, 1032), (8, 5461, 5461)])
@pytest.mark.parametrize("t", [1, 7])
def test_adam_rows(r, n, ldgc, t):
    GC, M, V = adam_inputs(r, n, 20, ldgc)
    if t == 1:
        M.zero_(); V.zero_()
    M0, V0 = to_f64(M).copy(), to_f64(V).copy()
    U = torch.full((r, n), float("nan"), device=DEV)
    grass.adam_rows(GC, M, V, LR, B1, B2, EPS, t, U)
    f = np.float32
    wU = ref.adam_rows(to_f64(GC), M0, V0, float(f(LR)), float(f(B1)), float(f(B2)), float(f(EPS)), t)
    assert rel_fro(to_f64(U), wU) <= TOL_F32
    assert rel_fro(to_f64(M), M0) <= TOL_F32
    assert rel_fro(to_f64(V), V0) <= TOL_F32
    np.testing.assert_allclose(to_f64(U), wU, rtol=5e-6, atol=1e-6 * LR)  # atol: m can cancel


@pytest.mark.parametrize("wdtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("m,n,r,dup,ldw", [(256, 256, 16, False, 256), (200, 1376, 64, True, 1376),
                                           (50, 333, 50, True, 333), (512, 1030, 100, True, 1040),
                                           (9, 5461, 4, False, 5461)])
def test_scatter_update_and_fused_adam_scatter(wdtype, m, n, r, dup, ldw):
    idx, rho = make_idx(m, r, 31, dup)
    d_idx, d_rho = torch.from_numpy(idx).to(DEV), torch.from_numpy(rho).to(DEV)
    alpha = 0.25
    W = randn((m, n), wdtype, 40, scale=0.02, ld=ldw)
    W0_bits = to_np(W).copy()
    W0 = to_f64(W).copy()
    GC, M, V = adam_inputs(r, n, 50, n)
    f = np.float32
    Mo, Vo = to_f64(M).copy(), to_f64(V).copy()
    wU = ref.adam_rows(to_f64(GC), Mo, Vo, float(f(LR)), float(f(B1)), float(f(B2)), float(f(EPS)), 3)

    # unfused: U from the GPU Adam, then scatter
    M1, V1, W1 = M.clone(), V.clone(), W.clone()
    U = torch.empty((r, n), device=DEV)
    grass.adam_rows(GC, M1, V1, LR, B1, B2, EPS, 3, U)
    grass.scatter_update(W1, d_idx, d_rho, alpha, U)
    # fused
    M2, V2, W2 = M.clone(), V.clone(), W.clone()
    grass.adam_scatter(GC, M2, V2, LR, B1, B2, EPS, 3, W2, d_idx, d_rho, alpha)

    Wo = W0.copy()
    ref.scatter_update(Wo, idx, rho, float(f(alpha)), wU)
    sel = np.unique(idx)
    rest = np.setdiff1d(np.arange(m), sel)
    for Wg, Mg, Vg in ((W1, M1, V1), (W2, M2, V2)):
        got = to_f64(Wg)
        assert rel_fro(got[sel], Wo[sel]) <= tol_for(wdtype)
        # the update itself (W's old value dominates the metric above)
        delta_tol = TOL_F32 if wdtype == torch.float32 else None
        if delta_tol:
            assert rel_fro(got[sel] - W0[sel], Wo[sel] - W0[sel]) <= 1e-4  # fp32 cancellation
        else:
            slack = 4 * 2.0 ** -24 * (np.abs(W0[sel]) + np.abs(Wo[sel] - W0[sel]))  # fp32 sum
            assert (np.abs(got[sel] - Wo[sel]) <= 0.501 * bf16_ulp(Wo[sel]) + slack).all()
        assert np.array_equal(to_np(Wg)[rest], W0_bits[rest])  # other rows untouched, bit for bit
        assert rel_fro(to_f64(Mg), Mo) <= TOL_F32 and rel_fro(to_f64(Vg), Vo) <= TOL_F32
    assert torch.equal(W1, W2) and torch.equal(M1, M2) and torch.equal(V1, V2)


def test_adam_scatter_empty():
    W = torch.zeros((4, 8), device=DEV)
    e = torch.zeros((0, 8), device=DEV)
    i = torch.zeros((0,), dtype=torch.int32, device=DEV)
    grass.adam_scatter(e, e.clone(), e.clone(), LR, B1, B2, EPS, 1, W, i, torch.zeros(0, device=DEV), 1.0)
    assert (W == 0).all()


# ------------------------------------------------------------------------------ large-tile GEMM path
@pytest.mark.parametrize("layout", [grass.DY_TxM, grass.DY_MxT])
@pytest.mark.parametrize("T,m,n,r,dup", [
    (1000, 700, 1376, 300, True),    # ragged T, n = 5*256 + 96, panel padded 300 -> 512
    (2048, 512, 512, 512, False),    # exact tiles, r = m
    (4100, 600, 264, 257, False),    # one row past a tile boundary, narrow n, T tail of 4 rows
    (96, 300, 512, 256, False),      # fewer K tiles than ring stages
])
def test_compressed_grad_large_tile_kernel(layout, T, m, n, r, dup):
    """The 256 x 256 load-to-LDS kernel, forced for shapes small enough for a full oracle."""
    grass.set_test_option(grass.TEST_GEMM_TILE, 256)
    dY = randn((T, m), torch.bfloat16, 11, scale=0.1)
    X = randn((T, n), torch.bfloat16, 12)
    idx, rho = make_idx(m, r, 13, dup)
    d_idx, d_rho = torch.from_numpy(idx).to(DEV), torch.from_numpy(rho).to(DEV)
    dY_dev = dY if layout == grass.DY_TxM else dY.t().contiguous()
    got = to_f64(gpu_cgrad(dY_dev, X, d_idx, d_rho, layout))
    want = ref.compressed_grad(to_np(dY), to_np(X), idx, rho)
    assert np.isfinite(got).all()
    assert rel_fro(got, want) <= 2e-5
    assert np.abs(got - want).max() <= 1e-4 * np.abs(want).max()


@pytest.mark.parametrize("T,m,n", [(1000, 520, 264), (2048, 512, 768)])
def test_dense_grad_large_tile_kernel(T, m, n):
    grass.set_test_option(grass.TEST_GEMM_TILE, 256)
    dY = randn((T, m), torch.bfloat16, 15, scale=0.1)
    X = randn((T, n), torch.bfloat16, 16)
    G = gpu_dense(dY, X, torch.float32)
    assert rel_fro(to_f64(G), ref.full_grad(to_np(dY), to_np(X))) <= 2e-5


def test_compressed_grad_large_tile_chosen_by_shape():
    """A shape for which the launcher picks the large tile by itself; the oracle is evaluated
    on a lattice of rows and columns that touches every 256 x 256 tile and every wavefront."""
    T, m, n, r = 8192 + 37, 2048, 2048, 1024
    dY = randn((T, m), torch.bfloat16, 21, scale=0.1)
    X = randn((T, n), torch.bfloat16, 22)
    idx, rho = make_idx(m, r, 23, False)
    got = to_f64(gpu_cgrad(dY, X, torch.from_numpy(idx).to(DEV), torch.from_numpy(rho).to(DEV)))
    rows = np.arange(5, r, 37)
    cols = np.arange(3, n, 29)
    want = ref.compressed_grad(to_np(dY), np.ascontiguousarray(to_np(X)[:, cols]), idx[rows], rho[rows])
    sub = got[np.ix_(rows, cols)]
    assert rel_fro(sub, want) <= 2e-5
    assert np.abs(sub - want).max() <= 1e-4 * np.abs(want).max()


# ------------------------------------------------------------------------------ fused refresh statistic
@pytest.mark.parametrize("dtype,layout,T,m,n,pad", [
    (torch.bfloat16, grass.DY_TxM, 1024, 512, 512, 0),     # fused: exact tiles
    (torch.bfloat16, grass.DY_TxM, 2048, 1032, 1376, 0),   # fused: ragged tiles in both dimensions
    (torch.bfloat16, grass.DY_TxM, 96, 264, 24, 8),        # fused: tiny n, padded leading dimensions
    (torch.bfloat16, grass.DY_TxM, 1000, 512, 512, 0),     # T not a multiple of 32: via fp32 G
    (torch.bfloat16, grass.DY_TxM, 512, 130, 333, 0),      # odd n: via fp32 G
    (torch.bfloat16, grass.DY_MxT, 512, 256, 256, 0),      # transposed storage: via fp32 G
    (torch.float32, grass.DY_TxM, 512, 256, 256, 0),       # fp32 inputs: via fp32 G
])
@pytest.mark.parametrize("force_fused", [True, False])
def test_grad_row_stats_without_storing_G(force_fused, dtype, layout, T, m, n, pad):
    """The fused form is chosen by itself only for layers with enough output tiles to fill
    the machine; here it is forced so that small shapes exercise it, and the same shapes also
    run the way the launcher would choose (fp32 G inside the workspace, then the statistic)."""
    if force_fused:
        grass.set_test_option(grass.TEST_FUSED_STATS, 1)
    dY = randn((T, m), dtype, 31, scale=0.1, ld=m + pad)
    X = randn((T, n), dtype, 32, ld=n + pad)
    dY_dev = dY if layout == grass.DY_TxM else dY.t().contiguous()
    out = torch.full((m,), float("nan"), device=DEV)
    dt = grass.F32 if dtype == torch.float32 else grass.BF16
    ldy = dY_dev.stride(0)
    ws = grass.workspace(grass.grad_row_stats_workspace(T, m, n, dt, layout, ldy, X.stride(0)))
    grass.grad_row_stats(dY_dev, X, out, ws, layout)
    want = ref.row_stats(ref.full_grad(to_np(dY), to_np(X)))
    got = to_f64(out)
    assert rel_fro(got, want) <= TOL_F32
    np.testing.assert_allclose(got, want, rtol=1e-5)


def test_grad_row_stats_small_workspace_is_enough_when_fused():
    """The point of the fused form: no m x n buffer.  4096 x 4096 needs well under 1 MB; a
    small layer (too few tiles to fill the machine without splitting K) keeps G in the workspace."""
    assert grass.grad_row_stats_workspace(131072, 4096, 4096, grass.BF16) < 1 << 20
    assert grass.grad_row_stats_workspace(131072, 4096, 4096, grass.F32) > 4096 * 4096 * 4
    assert grass.grad_row_stats_workspace(65536, 512, 512, grass.BF16) > 512 * 512 * 4


# ------------------------------------------------------------------------------ column projection
@pytest.mark.parametrize("wdtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("m,n,r,dup,ldw", [(64, 64, 8, False, 64), (200, 96, 40, True, 96),
                                           (333, 130, 130, True, 136), (1030, 512, 100, True, 512),
                                           (70, 5461, 300, True, 5461), (5, 9, 3, False, 9)])
def test_scatter_update_cols(wdtype, m, n, r, dup, ldw):
    idx, rho = make_idx(n, r, 61, dup)
    d_idx, d_rho = torch.from_numpy(idx).to(DEV), torch.from_numpy(rho).to(DEV)
    W = randn((m, n), wdtype, 62, scale=0.02, ld=ldw)
    W0 = to_f64(W).copy()
    W0_bits = to_np(W).copy()
    U = randn((r, m), torch.float32, 63, scale=1e-3).contiguous()
    grass.scatter_update_cols(W, d_idx, d_rho, 0.25, U)
    Wo = W0.copy()
    ref.scatter_update_cols(Wo, idx, rho, float(np.float32(0.25)), to_f64(U))
    got = to_f64(W)
    sel = np.unique(idx)
    assert rel_fro(got[:, sel], Wo[:, sel]) <= tol_for(wdtype)
    slack = 4 * 2.0 ** -24 * (np.abs(W0[:, sel]) + np.abs(Wo[:, sel] - W0[:, sel]))
    if wdtype == torch.bfloat16:
        assert (np.abs(got[:, sel] - Wo[:, sel]) <= 0.501 * bf16_ulp(Wo[:, sel]) + slack).all()
    else:
        assert (np.abs(got[:, sel] - Wo[:, sel]) <= 2.0 ** -23 * np.abs(Wo[:, sel]) + slack).all()
    rest = np.setdiff1d(np.arange(n), sel)
    assert np.array_equal(to_np(W)[:, rest], W0_bits[:, rest])  # other columns untouched


@pytest.mark.parametrize("T", [32, 64, 96, 128, 160, 192, 224, 256, 288, 1056])
def test_large_tile_kernel_every_pipeline_length(T):
    """1 to 9 and 33 K tiles per workgroup: prologue, steady state and drain of the LDS ring."""
    grass.set_test_option(grass.TEST_GEMM_TILE, 256)
    m, n, r = 300, 264, 260
    dY = randn((T, m), torch.bfloat16, 71, scale=0.1)
    X = randn((T, n), torch.bfloat16, 72)
    idx, rho = make_idx(m, r, 73, False)
    got = to_f64(gpu_cgrad(dY, X, torch.from_numpy(idx).to(DEV), torch.from_numpy(rho).to(DEV)))
    want = ref.compressed_grad(to_np(dY), to_np(X), idx, rho)
    assert rel_fro(got, want) <= 2e-5
    assert np.abs(got - want).max() <= 1e-4 * np.abs(want).max()


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("layout", [grass.DY_TxM, grass.DY_MxT])
@pytest.mark.parametrize("T,n,ms,rs,tile", [
    (512, 256, (256, 256, 256), (16, 16, 16), None),    # q, k, v of the small configuration
    (300, 150, (200, 90), (37, 13), None),              # nothing divides anything; r not a multiple of 8
    (1056, 264, (300, 520, 64), (130, 129, 0), "256"),  # large tile, an empty set in last place
    (777, 333, (130, 40, 50), (0, 40, 9), None),        # an empty set first, odd n
    (2048, 512, (384,), (260,), "256"),                 # a group of one
    (130, 64, (2048, 2056, 4096), (512, 600, 700), None),  # wide sets: each gathered through LDS
    (130, 64, (2048, 300), (512, 40), None),            # a wide set next to a narrow one: separate gathers
    (257, 72, (520, 264, 1376), (128, 40, 200), None),  # narrow sets: one gather launch for all
])
def test_compressed_grad_group_matches_per_matrix_oracle(dtype, layout, T, n, ms, rs, tile):
    """Several matrices sharing X (q, k, v): every output equals the single-matrix definition."""
    if tile:
        grass.set_test_option(grass.TEST_GEMM_TILE, int(tile))
    X = randn((T, n), dtype, 20)
    dYs, idxs, rhos, host = [], [], [], []
    for i, (m, r) in enumerate(zip(ms, rs)):
        dY = randn((T, m), dtype, 21 + i, scale=0.1)
        idx, rho = make_idx(m, r, 30 + i, duplicates=(i == 1))
        host.append((dY, idx, rho))
        dYs.append(dY if layout == grass.DY_TxM else dY.t().contiguous())
        idxs.append(torch.from_numpy(idx).to(DEV))
        rhos.append(torch.from_numpy(rho).to(DEV))
    GCs = [torch.full((r, n), float("nan"), dtype=torch.float32, device=DEV) for r in rs]
    dt = grass.F32 if dtype == torch.float32 else grass.BF16
    ws = grass.workspace(grass.cgrad_group_workspace(T, n, rs, dt, layout))
    grass.compressed_grad_group(dYs, X, idxs, rhos, GCs, ws, layout)
    for (dY, idx, rho), GC in zip(host, GCs):
        want = ref.compressed_grad(to_np(dY), to_np(X), idx, rho)
        got = to_f64(GC)
        assert got.shape == want.shape and np.isfinite(got).all()
        if want.size:
            assert rel_fro(got, want) <= 2e-5
            assert np.abs(got - want).max() <= 1e-4 * np.abs(want).max()


@pytest.mark.parametrize("tile", ["256", "128"])
@pytest.mark.parametrize("T,m,n,r,ldx,xoff", [
    (1056, 300, 531, 260, 531, 0),    # odd n: every other row of X starts in the middle of a word
    (1056, 300, 531, 260, 533, 2),    # odd leading dimension, X itself only 4-byte aligned
    (520, 300, 1365, 257, 1365, 0),   # the 5461-wide MLP of the 1B model, quartered
    (777, 130, 334, 129, 340, 0),     # even n that is not a multiple of 8
    (64, 40, 9, 40, 9, 0),            # fewer columns than one 16-byte chunk and a half
])
def test_compressed_grad_with_activations_that_break_16_byte_rows(tile, T, m, n, r, ldx, xoff):
    """X whose rows cannot be read in aligned 16-byte chunks is first copied into padded rows."""
    grass.set_test_option(grass.TEST_GEMM_TILE, int(tile))
    dY = randn((T, m), torch.bfloat16, 51, scale=0.1)
    flat = randn((1, T * ldx + xoff), torch.bfloat16, 52)[0]
    X = flat[xoff:xoff + T * ldx].view(T, ldx)[:, :n]
    assert X.data_ptr() % 4 == 0 and (xoff == 0 or X.data_ptr() % 16 != 0)
    idx, rho = make_idx(m, r, 53, False)
    got = to_f64(gpu_cgrad(dY, X, torch.from_numpy(idx).to(DEV), torch.from_numpy(rho).to(DEV)))
    want = ref.compressed_grad(to_np(dY), to_np(X), idx, rho)
    assert np.isfinite(got).all()
    assert rel_fro(got, want) <= 2e-5
    assert np.abs(got - want).max() <= 1e-4 * np.abs(want).max()


@pytest.mark.parametrize("T,m,n", [(1056, 301, 531), (520, 1365, 264), (96, 13, 9)])
def test_dense_grad_with_unaligned_widths_on_the_large_tile(T, m, n):
    """Full gradient when neither m nor n is a multiple of 8: dY goes through the packing
    pass with the identity selection, X through the aligning copy."""
    grass.set_test_option(grass.TEST_GEMM_TILE, 256)
    dY = randn((T, m), torch.bfloat16, 55, scale=0.1)
    X = randn((T, n), torch.bfloat16, 56)
    G = gpu_dense(dY, X, torch.float32)
    want = ref.full_grad(to_np(dY), to_np(X))
    assert rel_fro(to_f64(G), want) <= 2e-5
    ss = torch.empty(m, device=DEV)
    ws = grass.workspace(grass.grad_row_stats_workspace(T, m, n, grass.BF16, grass.DY_TxM, m, n))
    grass.grad_row_stats(dY, X, ss, ws)
    assert rel_fro(ss.cpu().numpy(), ref.row_stats(want)) <= TOL_F32


# ------------------------------------------------------------------------------ bf16 moments
@pytest.mark.parametrize("r,n,ldgc", [(16, 256, 256), (37, 1376, 1376), (5, 333, 333), (8, 5461, 5461)])
@pytest.mark.parametrize("t", [1, 7])
def test_adam_rows_with_bf16_moments(r, n, ldgc, t):
    """Moments stored in bf16: rounded once per step, the update taken from the stored values."""
    GC, M, V = adam_inputs(r, n, 60, ldgc)
    M, V = M.to(torch.bfloat16), V.to(torch.bfloat16)
    if t == 1:
        M.zero_(); V.zero_()
    M0, V0 = to_f64(M).copy(), to_f64(V).copy()
    Mold, Vold, g = M0.copy(), V0.copy(), to_f64(GC)
    U = torch.full((r, n), float("nan"), device=DEV)
    grass.adam_rows(GC, M, V, LR, B1, B2, EPS, t, U)
    f = np.float32
    wU = ref.adam_rows(to_f64(GC), M0, V0, float(f(LR)), float(f(B1)), float(f(B2)), float(f(EPS)), t,
                       state_bf16=True)
    gM, gV = to_f64(M), to_f64(V)
    # fp32 arithmetic before the rounding: a moment may land on the neighbouring bf16 value
    # when its exact value is within fp32 rounding of a tie (rare, one ulp); where the two
    # terms cancel, the fp32 error of the terms themselves is added
    for got, want, terms in ((gM, M0, np.abs(Mold) + np.abs(g)), (gV, V0, np.abs(Vold) + g * g)):
        off = got != want
        assert off.mean() <= 1e-3
        assert (np.abs(got - want) <= 1.01 * bf16_ulp(want) + 4 * 2.0 ** -24 * terms).all()
    same = (gM == M0) & (gV == V0)
    np.testing.assert_allclose(to_f64(U)[same], wU[same], rtol=5e-6, atol=1e-6 * LR)
    assert rel_fro(to_f64(U), wU) <= TOL_BF16


@pytest.mark.parametrize("wdtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("m,n,r,dup", [(200, 1376, 64, True), (50, 333, 50, True), (256, 256, 16, False)])
def test_fused_adam_scatter_with_bf16_moments(wdtype, m, n, r, dup):
    idx, rho = make_idx(m, r, 61, dup)
    d_idx, d_rho = torch.from_numpy(idx).to(DEV), torch.from_numpy(rho).to(DEV)
    W = randn((m, n), wdtype, 62, scale=0.02)
    GC, M, V = adam_inputs(r, n, 63, n)
    M, V = M.to(torch.bfloat16), V.to(torch.bfloat16)
    # unfused with the same state dtype, then fused: identical bits
    M1, V1, W1 = M.clone(), V.clone(), W.clone()
    U = torch.empty((r, n), device=DEV)
    grass.adam_rows(GC, M1, V1, LR, B1, B2, EPS, 3, U)
    grass.scatter_update(W1, d_idx, d_rho, 0.25, U)
    M2, V2, W2 = M.clone(), V.clone(), W.clone()
    grass.adam_scatter(GC, M2, V2, LR, B1, B2, EPS, 3, W2, d_idx, d_rho, 0.25)
    assert torch.equal(W1, W2) and torch.equal(M1, M2) and torch.equal(V1, V2)
    # and against the oracle
    f = np.float32
    Mo, Vo = to_f64(M).copy(), to_f64(V).copy()
    wU = ref.adam_rows(to_f64(GC), Mo, Vo, float(f(LR)), float(f(B1)), float(f(B2)), float(f(EPS)), 3,
                       state_bf16=True)
    Wo = to_f64(W).copy()
    ref.scatter_update(Wo, idx, rho, 0.25, wU)
    sel = np.unique(idx)
    assert rel_fro(to_f64(W2)[sel], Wo[sel]) <= tol_for(wdtype)
    assert rel_fro(to_f64(M2), Mo) <= 1e-4 and rel_fro(to_f64(V2), Vo) <= 1e-4
    rest = np.setdiff1d(np.arange(m), sel)
    assert np.array_equal(to_np(W2)[rest], to_np(W)[rest])


# ------------------------------------------------------------------------------ dY stored m x T
@pytest.mark.parametrize("pairs", [True, False])
@pytest.mark.parametrize("T", [32, 64, 96, 128, 160, 192, 224, 256, 320, 384, 448, 1056, 1088])
def test_row_gathering_gemm_every_pipeline_length(T, pairs):
    """dY stored m x T with T a whole number of K tiles: the large-tile kernel gathers the
    selected rows itself (no packing pass); prologue, steady loop and drain at every length.
    An even number of K tiles takes the form that loads 64 values of k per row and request
    (unless switched off), an odd one the form with one load per K tile."""
    grass.set_test_option(grass.TEST_GEMM_TILE, 256)
    if not pairs:
        grass.set_test_option(grass.TEST_NO_PAIRS, 1)
    m, n, r = 300, 264, 260
    dY = randn((T, m), torch.bfloat16, 71, scale=0.1)
    X = randn((T, n), torch.bfloat16, 72)
    idx, rho = make_idx(m, r, 73, True)
    dYt = dY.t().contiguous()
    got = to_f64(gpu_cgrad(dYt, X, torch.from_numpy(idx).to(DEV), torch.from_numpy(rho).to(DEV),
                           grass.DY_MxT))
    want = ref.compressed_grad(to_np(dY), to_np(X), idx, rho)
    assert np.isfinite(got).all()
    assert rel_fro(got, want) <= 2e-5
    assert np.abs(got - want).max() <= 1e-4 * np.abs(want).max()


@pytest.mark.parametrize("T,m,n,r,pad", [
    (2048, 1024, 512, 512, 0),     # exact tiles
    (1024, 5000, 520, 700, 0),     # rows spread over a tall matrix, 700 = 2 tiles + 188
    (512, 640, 1376, 257, 64),     # one row past a tile boundary, padded leading dimension
    (8192, 600, 264, 8, 0),        # a handful of rows, several K slices
    (16384 + 64, 520, 264, 300, 0),  # K slices of an odd number of K tiles, rounded up to pairs
])
def test_row_gathering_gemm_shapes_and_agreement_with_packing(T, m, n, r, pad):
    grass.set_test_option(grass.TEST_GEMM_TILE, 256)
    dYt = randn((m, T), torch.bfloat16, 75, scale=0.1, ld=T + pad)
    X = randn((T, n), torch.bfloat16, 76)
    idx, rho = make_idx(m, r, 77, False)
    d_idx, d_rho = torch.from_numpy(idx).to(DEV), torch.from_numpy(rho).to(DEV)
    got = gpu_cgrad(dYt, X, d_idx, d_rho, grass.DY_MxT)
    want = ref.compressed_grad(to_np(dYt), to_np(X), idx, rho, ref.DY_MxT)
    assert rel_fro(to_f64(got), want) <= 2e-5
    assert np.abs(to_f64(got) - want).max() <= 1e-4 * np.abs(want).max()
    # the packing path multiplies the same values in the same order inside a tile
    grass.set_test_option(grass.TEST_PACK_MXT, 1)
    packed = gpu_cgrad(dYt, X, d_idx, d_rho, grass.DY_MxT)
    assert rel_fro(to_f64(packed), want) <= 2e-5
    assert (got - packed).abs().max().item() <= 1e-5 * float(np.abs(want).max())


def test_dense_gradient_from_m_by_T_storage_without_packing():
    grass.set_test_option(grass.TEST_GEMM_TILE, 256)
    T, m, n = 1024, 520, 264
    dY = randn((T, m), torch.bfloat16, 78, scale=0.1)
    X = randn((T, n), torch.bfloat16, 79)
    G = gpu_dense(dY.t().contiguous(), X, torch.float32, grass.DY_MxT)
    assert rel_fro(to_f64(G), ref.full_grad(to_np(dY), to_np(X))) <= 2e-5


# ------------------------------------------------------------------------------ largest sizes
def test_most_rows_one_launch_takes():
    """r = 65535, the most rows the row-indexed launches take (a grid dimension): compressed
    gradient, Adam, scatter and the fused form against the oracle; r = 65536 is refused."""
    T, m, n, r = 64, 70000, 24, 65535
    dY = randn((T, m), torch.bfloat16, 91, scale=0.1)
    X = randn((T, n), torch.bfloat16, 92)
    idx, rho = make_idx(m, r, 93, False)
    d_idx, d_rho = torch.from_numpy(idx).to(DEV), torch.from_numpy(rho).to(DEV)
    GC = gpu_cgrad(dY, X, d_idx, d_rho)
    want = ref.compressed_grad(to_np(dY), to_np(X), idx, rho)
    assert rel_fro(to_f64(GC), want) <= 2e-5
    M = torch.zeros((r, n), device=DEV)
    V = torch.zeros((r, n), device=DEV)
    W = randn((m, n), torch.bfloat16, 94, scale=0.02)
    W0 = to_f64(W).copy()
    grass.adam_scatter(GC, M, V, LR, B1, B2, EPS, 1, W, d_idx, d_rho, 0.25)
    f = np.float32
    Mo, Vo = np.zeros((r, n)), np.zeros((r, n))
    U = ref.adam_rows(want, Mo, Vo, float(f(LR)), float(f(B1)), float(f(B2)), float(f(EPS)), 1)
    Wo = W0.copy()
    ref.scatter_update(Wo, idx, rho, 0.25, U)
    assert rel_fro(to_f64(W)[idx], Wo[idx]) <= TOL_BF16
    assert rel_fro(to_f64(M), Mo) <= TOL_F32 and rel_fro(to_f64(V), Vo) <= TOL_F32
    rest = np.setdiff1d(np.arange(m), idx)
    assert np.array_equal(to_f64(W)[rest], W0[rest])
    big = torch.zeros(65536, dtype=torch.int32, device=DEV)
    with pytest.raises(grass.GrassError) as e:
        grass.scatter_update(W, big, torch.ones(65536, device=DEV), 1.0, torch.zeros((65536, n), device=DEV))
    assert e.value.code == grass.ERR_SHAPE


def test_row_stats_and_selection_of_a_million_rows():
    m, n, r = 1 << 20, 8, 1500
    G = randn((m, n), torch.float32, 95)
    ss = torch.empty(m, device=DEV)
    grass.row_stats(G, ss)
    want = ref.row_stats(to_np(G))
    assert rel_fro(ss.cpu().numpy(), want) <= TOL_F32
    host = want.astype(np.float32)  # both sides select from the oracle's statistic
    ss = torch.from_numpy(host).to(DEV)
    for method, repl in [(grass.SEL_TOPR, False), (grass.SEL_MULTI_NORM, True), (grass.SEL_MULTI_NORM, False)]:
        idx, rho, status = gpu_select(ss, r, method, repl, seed=17, refresh_id=3)
        w_idx, w_rho, _ = ref.select_rows(host, r, method, repl, seed=17, refresh_id=3)
        assert status == grass.OK
        assert np.array_equal(idx.cpu().numpy(), w_idx), (method, repl)
        assert np.array_equal(rho.cpu().numpy(), w_rho)


def test_compressed_grad_group_too_large_for_a_joint_panel_runs_set_by_set():
    """Three sets whose joint slice of partial tiles would exceed the cached size: the group
    call falls back to one GEMM per set inside the same call.  Sampled rows against the oracle."""
    T, n, ms, rs = 512, 2048, (1100, 1300, 1100), (1024, 1024, 1000)
    X = randn((T, n), torch.bfloat16, 81)
    dYs, idxs, rhos, host = [], [], [], []
    for i, (m, r) in enumerate(zip(ms, rs)):
        dY = randn((T, m), torch.bfloat16, 82 + i, scale=0.1)
        idx, rho = make_idx(m, r, 86 + i, duplicates=False)
        host.append((dY, idx, rho))
        dYs.append(dY)
        idxs.append(torch.from_numpy(idx).to(DEV))
        rhos.append(torch.from_numpy(rho).to(DEV))
    GCs = [torch.full((r, n), float("nan"), dtype=torch.float32, device=DEV) for r in rs]
    ws = grass.workspace(grass.cgrad_group_workspace(T, n, rs, grass.BF16))
    grass.compressed_grad_group(dYs, X, idxs, rhos, GCs, ws)
    Xh = to_np(X)
    for (dY, idx, rho), GC in zip(host, GCs):
        assert torch.isfinite(GC).all()
        js = np.arange(1, len(idx), 67)
        want = ref.compressed_grad(to_np(dY), Xh, idx[js], rho[js])
        got = to_f64(GC)[js]
        assert rel_fro(got, want) <= 2e-5
        single = gpu_cgrad(dY, X, torch.from_numpy(idx).to(DEV), torch.from_numpy(rho).to(DEV))
        assert torch.equal(single, GC)  # the very same launches as the single call


# ------------------------------------------------------------------------------ seeded sweep of shapes
def _sweep_cases(count, seed):
    rng = np.random.default_rng(seed)
    cases = []
    for k in range(count):
        T = int(rng.choice([1, 7, 31, 32, 33, 64, 95, 128, 200, 257, 512, 700]))
        m = int(rng.integers(1, 600))
        n = int(rng.integers(1, 600))
        r = int(rng.integers(0, min(m, 300) + 1))
        pad_y, pad_x = int(rng.choice([0, 0, 3, 8])), int(rng.choice([0, 0, 5, 8]))
        layout = int(rng.integers(0, 2))
        tile = [None, "128", "256"][int(rng.integers(0, 3))]
        cases.append((k, T, m, n, r, pad_y, pad_x, layout, tile))
    return cases


@pytest.mark.parametrize("k,T,m,n,r,pad_y,pad_x,layout,tile", _sweep_cases(48, 2406))
def test_compressed_grad_and_dense_grad_shape_sweep(k, T, m, n, r, pad_y, pad_x, layout, tile):
    """Seeded random shapes, paddings, layouts and forced tiles: every combination of packing,
    aligning copy, K tail and tile kind the launcher can take."""
    if tile:
        grass.set_test_option(grass.TEST_GEMM_TILE, int(tile))
    X = randn((T, n), torch.bfloat16, 9000 + k, ld=n + pad_x)
    if layout == grass.DY_TxM:
        dY_dev = randn((T, m), torch.bfloat16, 9100 + k, scale=0.1, ld=m + pad_y)
        dY_host = to_np(dY_dev)
    else:
        dY_dev = randn((m, T), torch.bfloat16, 9100 + k, scale=0.1, ld=T + pad_y)
        dY_host = np.ascontiguousarray(to_np(dY_dev).T)
    idx, rho = make_idx(m, r, 9200 + k, duplicates=bool(k % 2))
    got = to_f64(gpu_cgrad(dY_dev, X, torch.from_numpy(idx).to(DEV), torch.from_numpy(rho).to(DEV), layout))
    want = ref.compressed_grad(dY_host, to_np(X), idx, rho)
    assert got.shape == want.shape and np.isfinite(got).all()
    if want.size:
        assert np.abs(got - want).max() <= 1e-4 * max(np.abs(want).max(), 1e-30) + 1e-30
    G = to_f64(gpu_dense(dY_dev, X, torch.float32, layout))
    wantG = ref.full_grad(dY_host, to_np(X))
    assert np.abs(G - wantG).max() <= 1e-4 * max(np.abs(wantG).max(), 1e-30) + 1e-30


def _update_cases(count, seed):
    rng = np.random.default_rng(seed)
    out = []
    for k in range(count):
        m = int(rng.integers(1, 400))
        n = int(rng.choice([1, 3, 4, 8, 63, 64, 100, 256, 333, 1024, 1031, 2052]))
        r = int(rng.integers(0, min(m, 150) + 1))
        out.append((k, m, n, r, int(rng.choice([0, 0, 1, 4])), bool(rng.integers(0, 2)),
                    [torch.float32, torch.bfloat16][int(rng.integers(0, 2))],
                    [torch.float32, torch.bfloat16][int(rng.integers(0, 2))]))
    return out


@pytest.mark.parametrize("k,m,n,r,pad,dup,wdtype,sdtype", _update_cases(32, 1766))
def test_adam_scatter_and_column_update_shape_sweep(k, m, n, r, pad, dup, wdtype, sdtype):
    """Seeded random shapes for the fused Adam + row update (both state dtypes) and for the
    column update: vector and element paths, padded leading dimensions, duplicate rows."""
    idx, rho = make_idx(m, r, 7000 + k, dup)
    d_idx, d_rho = torch.from_numpy(idx).to(DEV), torch.from_numpy(rho).to(DEV)
    W = randn((m, n), wdtype, 7100 + k, scale=0.02, ld=n + pad)
    W0, W0_bits = to_f64(W).copy(), to_np(W).copy()
    GC, M, V = adam_inputs(r, n, 7200 + k, n + pad) if r else (torch.zeros((0, n), device=DEV),) * 3
    M, V = M.to(sdtype).contiguous(), V.to(sdtype).contiguous()
    Mo, Vo = to_f64(M).copy(), to_f64(V).copy()
    grass.adam_scatter(GC, M, V, LR, B1, B2, EPS, 2, W, d_idx, d_rho, 0.25)
    f = np.float32
    U = ref.adam_rows(to_f64(GC), Mo, Vo, float(f(LR)), float(f(B1)), float(f(B2)), float(f(EPS)), 2,
                      state_bf16=sdtype == torch.bfloat16)
    Wo = W0.copy()
    ref.scatter_update(Wo, idx, rho, 0.25, U)
    sel = np.unique(idx)
    if len(sel):
        assert rel_fro(to_f64(W)[sel], Wo[sel]) <= tol_for(wdtype)
        assert rel_fro(to_f64(M), Mo) <= (1e-2 if sdtype == torch.bfloat16 else TOL_F32)
        assert rel_fro(to_f64(V), Vo) <= (1e-2 if sdtype == torch.bfloat16 else TOL_F32)
    rest = np.setdiff1d(np.arange(m), sel)
    assert np.array_equal(to_np(W)[rest], W0_bits[rest])
    # column form on the transposed weight: W2 is n x m, columns idx of it are updated
    if n <= 1100:
        W2 = randn((n, m), wdtype, 7300 + k, scale=0.02, ld=m + pad)
        W2o, W2_bits = to_f64(W2).copy(), to_np(W2).copy()
        U32 = torch.from_numpy(U.astype(np.float32)).to(DEV).contiguous()
        grass.scatter_update_cols(W2, d_idx, d_rho, 0.25, U32)
        ref.scatter_update_cols(W2o, idx, rho, 0.25, U.astype(np.float32).astype(np.float64))
        got = to_f64(W2)
        if len(sel):
            assert rel_fro(got[:, sel], W2o[:, sel]) <= tol_for(wdtype)
        assert np.array_equal(to_np(W2)[:, rest], W2_bits[:, rest])


@pytest.mark.parametrize("case", range(24))
def test_select_rows_random_sizes_bit_exact(case):
    rng = np.random.default_rng(4100 + case)
    m = int(rng.choice([1, 2, 63, 64, 65, 100, 1000, 4095, 4096, 4097, 20000, 70001]))
    method, repl = METHODS[case % len(METHODS)]
    with_repl = repl and method != grass.SEL_TOPR
    r = int(rng.integers(0, 2000)) if with_repl else int(rng.integers(0, min(m, 2000) + 1))
    ss = sumsq_case(m, ["chi2", "lognormal", "ties", "wide"][case % 4], 4200 + case)
    idx, rho, status = gpu_select(torch.from_numpy(ss).to(DEV), r, method, repl, seed=case, refresh_id=case * 7)
    w_idx, w_rho, _ = ref.select_rows(ss, r, method, repl, seed=case, refresh_id=case * 7)
    assert status == grass.OK
    assert np.array_equal(idx.cpu().numpy(), w_idx) and np.array_equal(rho.cpu().numpy(), w_rho)


# ------------------------------------------------------------------------------ the whole regular step in one call
@pytest.mark.parametrize("dtype,wdtype,sdtype", [(torch.bfloat16, torch.bfloat16, torch.float32),
                                                 (torch.bfloat16, torch.float32, torch.bfloat16),
                                                 (torch.float32, torch.float32, torch.float32)])
@pytest.mark.parametrize("T,n,ms,rs,want_gc,tile", [
    (512, 256, (256,), (16,), True, None),                   # one layer, G_C requested
    (4096, 512, (300, 520, 64), (130, 129, 0), False, None), # group, several K slices, an empty set
    (1056, 264, (300, 520), (130, 129), True, "256"),        # large tile, K tail
    (777, 334, (130, 90), (40, 9), False, None),             # n % 4 != 0: the tail on single elements
    (640, 1024, (400,), (256,), False, "256"),               # duplicates walk runs across the tile
])
def test_step_group_equals_the_separate_calls_and_the_oracle(dtype, wdtype, sdtype, T, n,
                                                             ms, rs, want_gc, tile):
    run_step_group(dtype, wdtype, sdtype, T, n, ms, rs, want_gc, tile)


@pytest.mark.parametrize("wdtype,sdtype", [(torch.bfloat16, torch.float32), (torch.float32, torch.bfloat16),
                                           (torch.bfloat16, torch.bfloat16), (torch.float32, torch.float32)])
@pytest.mark.parametrize("T,n,ms,rs,want_gc,tile", [
    (8192, 256, (300,), (40,), True, None),                  # one layer, 16 slices
    (8192, 256, (300, 520, 64), (40, 33, 8), False, None),   # a group of three in one launch
    (8192, 1280, (24,), (40,), False, None),                 # every row drawn repeatedly; five column blocks
    (8192, 264, (300, 90), (40, 9), True, None),             # the last column block is mostly empty
    (8192, 1024, (400,), (256,), True, "256"),               # large tile: 32 slices
    (8200, 512, (300,), (200,), False, "256"),               # ... with a ragged last K tile
    (4608, 256, (64,), (9,), False, None),                   # the fewest slices that take this kernel (9)
    (6656, 128, (64,), (5,), True, None),                    # 13 slices: quarters of 4, 4, 4 and 1
    (5120, 128, (40,), (8,), False, None),                   # 10 slices: quarters of 3, 3, 3 and 1
])
def test_step_group_with_more_than_eight_k_slices(wdtype, sdtype, T, n, ms, rs, want_gc, tile):
    """Short, wide products (the layers of the small models at their token batch) split K into
    dozens of slices; the step's tail is then the kernel whose four wavefronts each add a quarter
    of the slices and meet in LDS.  The plan query confirms that these shapes take it."""
    if tile:
        grass.set_test_option(grass.TEST_GEMM_TILE, int(tile))
    total = sum((r + 7) // 8 * 8 for r in rs) if len(rs) > 1 else rs[0]
    assert grass.cgrad_plan(T, n, total, grass.BF16)[1] > 8
    run_step_group(torch.bfloat16, wdtype, sdtype, T, n, ms, rs, want_gc, tile)


def run_step_group(dtype, wdtype, sdtype, T, n, ms, rs, want_gc, tile):
    if tile:
        grass.set_test_option(grass.TEST_GEMM_TILE, int(tile))
    X = randn((T, n), dtype, 120)
    dYs, idxs, rhos, Ms, Vs, Ws, host = [], [], [], [], [], [], []
    for i, (m, r) in enumerate(zip(ms, rs)):
        dY = randn((T, m), dtype, 121 + i, scale=0.1)
        idx, rho = make_idx(m, r, 130 + i, duplicates=True)
        GC_, M, V = adam_inputs(r, n, 140 + i, n) if r else (None, torch.zeros((0, n), device=DEV),
                                                             torch.zeros((0, n), device=DEV))
        M, V = M.to(sdtype).contiguous(), V.to(sdtype).contiguous()
        W = randn((m, n), wdtype, 150 + i, scale=0.02)
        host.append((dY, idx, rho, to_f64(M).copy(), to_f64(V).copy(), to_f64(W).copy(), to_np(W).copy()))
        dYs.append(dY); idxs.append(torch.from_numpy(idx).to(DEV)); rhos.append(torch.from_numpy(rho).to(DEV))
        Ms.append(M); Vs.append(V); Ws.append(W)
    GCs = [torch.full((r, n), float("nan"), device=DEV) for r in rs] if want_gc else None
    dt = grass.F32 if dtype == torch.float32 else grass.BF16
    ws = grass.workspace(grass.step_group_workspace(T, n, rs, dt))
    grass.step_group(dYs, X, idxs, rhos, Ms, Vs, Ws, LR, B1, B2, EPS, 3, 0.25, ws, GCs=GCs)
    f = np.float32
    for i, (dY, idx, rho, M0, V0, W0, W0_bits) in enumerate(host):
        if rs[i] == 0:
            assert np.array_equal(to_np(Ws[i]), W0_bits)
            continue
        GC = ref.compressed_grad(to_np(dY), to_np(X), idx, rho)
        if want_gc:
            assert rel_fro(to_f64(GCs[i]), GC) <= 2e-5
        U = ref.adam_rows(GC, M0, V0, float(f(LR)), float(f(B1)), float(f(B2)), float(f(EPS)), 3,
                          state_bf16=sdtype == torch.bfloat16)
        Wo = W0.copy()
        ref.scatter_update(Wo, idx, rho, 0.25, U)
        sel = np.unique(idx)
        state_tol = 1e-2 if sdtype == torch.bfloat16 else 2e-5
        assert rel_fro(to_f64(Ms[i]), M0) <= state_tol and rel_fro(to_f64(Vs[i]), V0) <= state_tol
        assert rel_fro(to_f64(Ws[i])[sel], Wo[sel]) <= tol_for(wdtype)
        rest = np.setdiff1d(np.arange(ms[i]), sel)
        assert np.array_equal(to_np(Ws[i])[rest], W0_bits[rest])


@pytest.mark.parametrize("layout", [grass.DY_TxM, grass.DY_MxT])
def test_compressed_grad_very_long_token_batch(layout):
    """T = 300001 (beyond the paper's 262144 tokens per step): launch grids indexed by t stay legal."""
    T, m, n, r = 300001, 72, 64, 9
    dY = randn((T, m), torch.bfloat16, 171, scale=0.1)
    X = randn((T, n), torch.bfloat16, 172)
    idx, rho = make_idx(m, r, 173, False)
    dY_dev = dY if layout == grass.DY_TxM else dY.t().contiguous()
    got = to_f64(gpu_cgrad(dY_dev, X, torch.from_numpy(idx).to(DEV), torch.from_numpy(rho).to(DEV), layout))
    want = ref.compressed_grad(to_np(dY), to_np(X), idx, rho)
    assert rel_fro(got, want) <= 2e-5


@pytest.mark.parametrize("layout,T", [(grass.DY_TxM, 4_200_003), (grass.DY_MxT, 4_200_003),
                                      (grass.DY_MxT, 16_800_008)])
def test_compressed_grad_millions_of_tokens(layout, T):
    """More than 65535 blocks of t in every packing kernel (64 and 256 rows of t per block): the
    block index over t is the x dimension of their grids."""
    m, n, r = 16, 8, 4
    dY = randn((T, m), torch.bfloat16, 181, scale=0.1)
    X = randn((T, n), torch.bfloat16, 182)
    idx, rho = make_idx(m, r, 183, False)
    dY_dev = dY if layout == grass.DY_TxM else dY.t().contiguous()
    got = to_f64(gpu_cgrad(dY_dev, X, torch.from_numpy(idx).to(DEV), torch.from_numpy(rho).to(DEV), layout))
    want = ref.compressed_grad(to_np(dY), to_np(X), idx, rho)
    assert rel_fro(got, want) <= 2e-5


@pytest.mark.parametrize("T,m,n,r,dup,pad,shift", [
    (257, 1024, 64, 64, False, 0, 0),      # smallest shape that takes the staged gather; odd T
    (257, 1016, 64, 64, False, 0, 0),      # one step narrower / (next) one selected row fewer: plain
    (257, 1024, 64, 56, False, 0, 0),
    (130, 5464, 72, 600, True, 8, 0),      # row length not a power of two, padded rows, duplicates
    (131, 5461, 72, 600, True, 0, 0),      # odd row length: every row starts at another byte offset
    (67, 12288, 64, 1500, True, 0, 0),     # the longest rows staged two at a time
    (65, 12296, 64, 700, False, 0, 0),     # one step longer: one row per workgroup
    (34, 32760, 64, 900, True, 0, 0),      # the longest rows that are staged at all (64 KB of LDS)
    (33, 32768, 64, 600, False, 3, 0),     # one step longer: the plain gather
    (96, 4096, 128, 1024, False, 8, 1),    # rows that start 2 bytes after a 16-byte boundary
    (96, 4099, 128, 1024, True, 2, 5),     # odd everything
    (1, 4096, 64, 512, False, 0, 0),       # a single row of t
    (2, 2051, 64, 300, False, 0, 3),       # the first and the last vector of the matrix are partial
])
def test_compressed_grad_gather_staged_through_lds(T, m, n, r, dup, pad, shift):
    """Wide T x m gradients: the gather copies whole rows of dY into LDS first.  Shapes on both
    sides of every condition of that route (width, row length, alignment), against the oracle."""
    buf = randn((T, m + pad + shift), torch.bfloat16, 191, scale=0.1)
    dY = buf[:, shift:shift + m]
    X = randn((T, n), torch.bfloat16, 192)
    idx, rho = make_idx(m, r, 193, dup)
    got = to_f64(gpu_cgrad(dY, X, torch.from_numpy(idx).to(DEV), torch.from_numpy(rho).to(DEV)))
    want = ref.compressed_grad(np.ascontiguousarray(to_np(dY)), to_np(X), idx, rho)
    assert rel_fro(got, want) <= 2e-5


@pytest.mark.parametrize("sdtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("T,m,n,r,dup,want_gc,tile", [
    (8192, 256, 64, 24, True, True, None),       # 16 slices, duplicates
    (8192, 1280, 96, 40, False, False, None),    # five column blocks
    (8192, 1024, 300, 256, True, False, "256"),  # large tile: 32 slices
    (4608, 264, 40, 9, False, True, None),       # the fewest slices that take this kernel
])
def test_step_cols_with_more_than_eight_k_slices(sdtype, T, m, n, r, dup, want_gc, tile):
    """The column-form step when K is split into more than eight slices: reduction and Adam run
    in the kernel that spreads the slices over its wavefronts, writing Adam's output to U."""
    if tile:
        grass.set_test_option(grass.TEST_GEMM_TILE, int(tile))
    assert grass.cgrad_plan(T, m, r, grass.BF16)[1] > 8
    run_step_cols(torch.bfloat16, sdtype, T, m, n, r, dup, want_gc, tile)


@pytest.mark.parametrize("sdtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("T,m,n,r,dup,want_gc,tile", [
    (512, 688, 256, 64, True, True, None),      # gate/up-shaped, duplicates
    (300, 130, 50, 17, False, False, None),     # nothing divides anything (m % 4 != 0: the tail on single elements)
    (1056, 520, 264, 260, True, False, "256"),  # large tile
    (4096, 64, 32, 8, False, True, None),       # several K slices for a small output
])
def test_step_cols_equals_the_separate_calls_and_the_oracle(sdtype, T, m, n, r, dup, want_gc, tile):
    """The column-form step in one call against the oracle (compressed gradient of the exchanged
    operands, Adam on r x m, update of r columns of W)."""
    run_step_cols(torch.bfloat16, sdtype, T, m, n, r, dup, want_gc, tile)


def test_step_cols_fp32_inputs():
    run_step_cols(torch.float32, torch.float32, 300, 130, 50, 17, True, True, None)


def run_step_cols(dtype, sdtype, T, m, n, r, dup, want_gc, tile):
    if tile:
        grass.set_test_option(grass.TEST_GEMM_TILE, int(tile))
    dY = randn((T, m), dtype, 201, scale=0.1)
    X = randn((T, n), dtype, 202)
    idx, rho = make_idx(n, r, 203, dup)
    d_idx, d_rho = torch.from_numpy(idx).to(DEV), torch.from_numpy(rho).to(DEV)
    _, M, V = adam_inputs(r, m, 204, m)
    M, V = M.to(sdtype).contiguous(), V.to(sdtype).contiguous()
    M0, V0 = to_f64(M).copy(), to_f64(V).copy()
    W = randn((m, n), torch.bfloat16, 207, scale=0.02)
    W0, W0_bits = to_f64(W).copy(), to_np(W).copy()
    U = torch.full((r, m), float("nan"), device=DEV)
    GC = torch.full((r, m), float("nan"), device=DEV) if want_gc else None
    dt = grass.F32 if dtype == torch.float32 else grass.BF16
    ws = grass.workspace(max(grass.step_cols_workspace(T, m, n, r, dt), 16))
    grass.step_cols(dY, X, d_idx, d_rho, M, V, U, W, LR, B1, B2, EPS, 3, 0.25, ws, GC=GC)
    f = np.float32
    want_gc_ref = ref.compressed_grad(to_np(X), to_np(dY), idx, rho)  # r x m
    if want_gc:
        assert rel_fro(to_f64(GC), want_gc_ref) <= 2e-5
    Uo = ref.adam_rows(want_gc_ref, M0, V0, float(f(LR)), float(f(B1)), float(f(B2)), float(f(EPS)), 3,
                       state_bf16=sdtype == torch.bfloat16)
    Wo = W0.copy()
    ref.scatter_update_cols(Wo, idx, rho, 0.25, Uo)
    state_tol = 1e-2 if sdtype == torch.bfloat16 else 2e-5
    assert rel_fro(to_f64(M), M0) <= state_tol and rel_fro(to_f64(V), V0) <= state_tol
    # U = -lr m^ / (sqrt(v^) + eps): with fp32 moments it carries the relative error of G_C and
    # a few fp32 roundings; with bf16 moments the oracle rounds the same values the same way, and
    # what is left is the rare element whose moment falls on the other side of a rounding boundary
    assert rel_fro(to_f64(U), Uo) <= (5e-2 if sdtype == torch.bfloat16 else 2e-5)
    sel = np.unique(idx)
    assert rel_fro(to_f64(W)[:, sel], Wo[:, sel]) <= TOL_BF16
    rest = np.setdiff1d(np.arange(n), sel)
    assert np.array_equal(to_np(W)[:, rest], W0_bits[:, rest])


def test_step_group_timing_hooks_change_nothing_but_fill_the_events():
    """grass_step_group_timed: the same step bit for bit, and two intervals that are positive and
    ordered (the matrix multiply ends before the fused tail starts)."""
    T, n, m, r = 4096, 512, 300, 130
    X = randn((T, n), torch.bfloat16, 300)
    dY = randn((T, m), torch.bfloat16, 301, scale=0.1)
    idx, rho = make_idx(m, r, 302, duplicates=True)
    d_idx, d_rho = torch.from_numpy(idx).to(DEV), torch.from_numpy(rho).to(DEV)
    ws = grass.workspace(grass.step_group_workspace(T, n, [r], grass.BF16))
    out = []
    for timed in (False, True):
        _, M, V = adam_inputs(r, n, 303, n)
        W = randn((m, n), torch.bfloat16, 304, scale=0.02)
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(4)]
        for e in ev:
            e.record()
        kw = dict(gemm_events=(ev[0], ev[1]), tail_events=(ev[2], ev[3])) if timed else {}
        grass.step_group([dY], X, [d_idx], [d_rho], [M], [V], [W], LR, B1, B2, EPS, 2, 0.25, ws, **kw)
        torch.cuda.synchronize()
        if timed:
            assert 0 < ev[0].elapsed_time(ev[1]) < 50 and 0 < ev[2].elapsed_time(ev[3]) < 50
            assert ev[1].elapsed_time(ev[2]) >= 0
        out.append((M, V, W))
    for a, b in zip(*out):
        assert torch.equal(a, b)
