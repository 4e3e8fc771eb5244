"""Reductions of one to sixteen K slices: every count of loads that the kernels issue together, and the turns behind
them, in the split-K sum, the fused tail of a step (rows on 16-byte boundaries and not) and its column form, against
64-bit products.  Bound: products of bf16 values are exact in fp32, sums of T of them off by about
sqrt(T) * 2^-24 = 4e-6; TOL_F32 (1e-5) covers it."""
import pytest
import torch

from paper_2406_17660_amd import grass
from gpu_util import DEV, TOL_F32

pytestmark = pytest.mark.gpu
BF = torch.bfloat16


def _rel(got, want):
    return float((got.double() - want).norm() / want.norm())


@pytest.mark.parametrize("n", [264, 261])
@pytest.mark.parametrize("slices", [*range(1, 10), 13, 16])
def test_every_number_of_slices(slices, n):
    T, m, r = 32 * 8 * slices, 264, 40  # eight K tiles of 32 tokens per slice
    grass.set_test_option(grass.TEST_GEMM_TILE, 256)
    grass.set_test_option(grass.TEST_MAX_K_SLICES, slices)
    assert grass.cgrad_plan(T, n, r, grass.BF16)[1] in (slices, slices - 1)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(slices)
    dY, X = (torch.randn(T, w, generator=gen, device=DEV).to(BF) for w in (m, n))
    W = torch.randn(m, n, generator=gen, device=DEV).to(BF)
    idx = torch.randperm(m, generator=gen, device=DEV)[:r].sort()[0].to(torch.int32)
    rho = torch.rand(r, generator=gen, device=DEV) + 0.5
    full = dY.double().t() @ X.double()
    G = torch.full((m, n), float("nan"), device=DEV)
    grass.dense_grad(dY, X, G, grass.workspace(grass.dense_workspace(T, m, n, grass.BF16)))
    assert _rel(G, full) <= TOL_F32
    want = rho.double()[:, None] * full[idx.long()]
    M, V = torch.zeros(r, n, device=DEV), torch.zeros(r, n, device=DEV)
    GC = torch.full((r, n), float("nan"), device=DEV)
    ws = grass.workspace(grass.step_group_workspace(T, n, [r], grass.BF16))
    grass.step_group([dY], X, [idx], [rho], [M], [V], [W], 1e-3, 0.9, 0.999, 1e-8, 1, 0.25, ws, GCs=[GC])
    assert _rel(GC, want) <= TOL_F32 and _rel(M, 0.1 * want) <= TOL_F32
    if n % 8 == 0:  # columns of an m x n weight: the transposed problem
        M, V, U = (torch.zeros(r, m, device=DEV) for _ in range(3))
        GC = torch.full((r, m), float("nan"), device=DEV)
        cols = torch.arange(r, dtype=torch.int32, device=DEV) * 6
        ws = grass.workspace(grass.step_cols_workspace(T, m, n, r, grass.BF16))
        grass.step_cols(dY, X, cols, rho, M, V, U, W, 1e-3, 0.9, 0.999, 1e-8, 1, 0.25, ws, GC=GC)
        want = rho.double()[:, None] * full.t()[cols.long()]
        assert _rel(GC, want) <= TOL_F32 and _rel(M, 0.1 * want) <= TOL_F32
