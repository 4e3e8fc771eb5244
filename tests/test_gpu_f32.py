"""GPU parity of the fp32 matrix-core product: tile edges, ragged tokens, K slices with and without a
workspace, groups, unaligned operands and subnormal inputs, against the fp64 oracle.

Bound: a sum of T products in fp32, whatever its order, is off by at most T * 2^-24 * sum |a b|; over
normal inputs the relative error grows like sqrt(T) * 2^-24, 6e-6 at the largest T here.  TOL_F32
(1e-5) covers it."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_2406_17660_amd import grass
from gpu_util import DEV, TOL_F32, rel_fro, to_f64, to_np

pytestmark = pytest.mark.gpu


def _inputs(T, m, n, r, layout, seed=0, shift=0):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    flat = torch.randn(T * m + shift, generator=g, device=DEV)[shift:]
    dY = flat.view(m, T) if layout == grass.DY_MxT else flat.view(T, m)
    X = torch.randn(T * n + shift, generator=g, device=DEV)[shift:].view(T, n)
    idx = torch.randint(0, m, (r,), generator=g, device=DEV).sort()[0].to(torch.int32)
    rho = torch.rand(r, generator=g, device=DEV) + 0.5
    return dY, X, idx, rho


def _want(dY, X, idx, rho, layout):
    d = to_f64(dY)
    return ref.compressed_grad(np.ascontiguousarray(d.T) if layout == grass.DY_MxT else d, to_f64(X),
                               to_np(idx), to_np(rho))


@pytest.mark.parametrize("tile", [64, 128])
@pytest.mark.parametrize("layout", [grass.DY_TxM, grass.DY_MxT])
@pytest.mark.parametrize("T,m,n,r,shift", [
    (1, 5, 1, 1, 0), (15, 70, 63, 63, 1), (16, 64, 64, 64, 0), (17, 200, 130, 65, 0),
    (1023, 140, 129, 129, 0), (1024, 96, 68, 3, 0), (2513, 300, 257, 130, 3), (4096, 128, 128, 128, 0)])
def test_product_at_tile_edges(tile, layout, T, m, n, r, shift):
    dY, X, idx, rho = _inputs(T, m, n, r, layout, shift=shift)
    want = _want(dY, X, idx, rho, layout)
    grass.set_test_option(grass.TEST_GEMM_TILE, tile)
    need = grass.cgrad_workspace(T, m, n, r, grass.F32, layout)
    for nbytes in (need, need // 2):  # fewer slices, or none, when the workspace is short
        GC = torch.full((r, n), float("nan"), device=DEV)
        grass.compressed_grad(dY, X, idx, rho, GC, grass.workspace(nbytes) if nbytes else None, layout)
        assert rel_fro(to_np(GC), want) <= TOL_F32
    G = torch.full((m, n), float("nan"), device=DEV)
    grass.dense_grad(dY, X, G, grass.workspace(grass.dense_workspace(T, m, n, grass.F32, layout)), layout)
    d = to_f64(dY)
    assert rel_fro(to_np(G), (d if layout == grass.DY_MxT else d.T) @ to_f64(X)) <= TOL_F32


@pytest.mark.parametrize("n", [48, 50])  # fused tail on 16-byte accesses, and on single elements
def test_group_step_equals_separate_calls(n):
    T, ms, rs = 1500, (70, 64, 9), (33, 64, 1)
    X = torch.randn(T, n, device=DEV)
    sets, GCs = [], []
    for k, (m, r) in enumerate(zip(ms, rs)):
        dY, _, idx, rho = _inputs(T, m, n, r, grass.DY_TxM, seed=k)
        idx = torch.randperm(m, device=DEV)[:r].sort()[0].to(torch.int32)
        sets.append((dY, idx, rho, torch.zeros(r, n, device=DEV), torch.zeros(r, n, device=DEV),
                     torch.zeros(m, n, device=DEV)))
        GCs.append(torch.full((r, n), float("nan"), device=DEV))
    ws = grass.workspace(grass.step_group_workspace(T, n, rs, grass.F32))
    dYs, idxs, rhos, Ms, Vs, Ws = (list(t) for t in zip(*sets))
    grass.step_group(dYs, X, idxs, rhos, Ms, Vs, Ws, 1e-3, 0.9, 0.999, 1e-8, 1, 0.5, ws, GCs=GCs)
    for dY, idx, rho, M, V, W, GC in zip(dYs, idxs, rhos, Ms, Vs, Ws, GCs):
        want = _want(dY, X, idx, rho, grass.DY_TxM)
        assert rel_fro(to_np(GC), want) <= TOL_F32
        assert rel_fro(to_np(M), 0.1 * want) <= TOL_F32
        # W started at 0: its selected rows are alpha * rho * U of the state that was stored
        U = -1e-3 * (to_f64(M) / 0.1) / (np.sqrt(to_f64(V) / 0.001) + 1e-8)
        rows = to_np(W)[to_np(idx)]
        assert rel_fro(rows, 0.5 * to_f64(rho)[:, None] * U) <= TOL_F32


def test_subnormal_inputs_and_nonfinite_neighbours():
    """Products of subnormal inputs are kept, and an Inf in a column or token that an output does not
    depend on does not reach it (edges are loaded twice or cleared, never multiplied by Inf)."""
    T, m, n = 33, 5, 6
    dY, X = torch.full((T, m), 1e-39, device=DEV), torch.full((T, n), 8.0, device=DEV)
    dY[:, 0] = float("inf")
    X[T - 1, 0] = float("inf")
    idx = torch.tensor([1, 3], dtype=torch.int32, device=DEV)
    GC = torch.empty(2, n, device=DEV)
    grass.compressed_grad(dY, X, idx, torch.ones(2, device=DEV), GC, None)
    got = to_np(GC)
    assert np.isinf(got[:, 0]).all()
    # 33 * 8e-39, in units of the smallest subnormal (1.4e-45): exact to a few of them
    assert np.abs(got[:, 1:].astype(np.float64) - 33 * 8 * float(np.float32(1e-39))).max() < 64 * 2.0 ** -149
