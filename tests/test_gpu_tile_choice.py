"""Which matrix-multiply kernel the launcher chooses where the choice costs most, and that every tile the chooser may
run on the K slices of either plan gives the oracle's sums."""
import pytest
import torch

from paper_2406_17660_amd import grass
from gpu_util import DEV

pytestmark = pytest.mark.gpu
BF = torch.bfloat16


@pytest.mark.parametrize("kernel,T,m,n,r", [
    # the large tile would copy an odd-width X: packed dY and the small tile on X in place
    (grass.KERNEL_128_STAGED, 41408, 680, 4109, 42), (grass.KERNEL_128_STAGED, 27488, 88, 439, 40),
    # short products: the pack and the tile that starts soonest
    (grass.KERNEL_128, 864, 240, 64, 58), (grass.KERNEL_128, 928, 1544, 136, 96),
    # rows gathered by the tile loads
    (grass.KERNEL_256_ROWS, 16384, 1024, 4096, 1024), (grass.KERNEL_256_ROWS, 8192, 2048, 2060, 1024)])
def test_tile_of_products_stored_mxt(kernel, T, m, n, r):
    dY, X = torch.zeros(m, T, dtype=BF, device=DEV), torch.zeros(T, n, dtype=BF, device=DEV)
    idx, rho, GC = torch.arange(r, dtype=torch.int32, device=DEV), torch.ones(r, device=DEV), torch.empty(r, n, device=DEV)
    grass.compressed_grad(dY, X, idx, rho, GC, grass.workspace(grass.cgrad_workspace(T, m, n, r, grass.BF16, grass.DY_MxT)),
                          grass.DY_MxT)
    assert grass.last_kernel() == kernel


@pytest.mark.parametrize("layout", [grass.DY_TxM, grass.DY_MxT])
@pytest.mark.parametrize("T", [32, 33, 63, 64, 96, 127, 1001, 1056, 2080, 2112, 2477])
def test_every_tile_on_slices_planned_for_the_large_one(T, layout):
    """Slices in units of 32 tokens (pairs of them for gathered rows), a ragged last one: the tiles
    give the same bits, those of a sum of all tokens.  Inf lies behind the last token and the last column."""
    m, n, r = 520, 504, 500
    gen = torch.Generator(device=DEV)
    gen.manual_seed(T)
    pad = -T % 8
    X = torch.full((T + 40, n + 8), float("inf"), dtype=BF, device=DEV)[:T, :n]
    X.copy_(torch.randn(T, n, generator=gen, device=DEV))
    dY = torch.full((T + 40, m + 8), float("inf"), dtype=BF, device=DEV)[:T, :m] if layout == grass.DY_TxM else \
        torch.full((m, T + pad + 64), float("inf"), dtype=BF, device=DEV)[:, :T]
    dY.copy_(torch.randn(dY.shape, generator=gen, device=DEV))
    idx = torch.randperm(m, generator=gen, device=DEV)[:r].sort()[0].to(torch.int32)
    rho = torch.rand(r, generator=gen, device=DEV) + 0.5
    rows = dY.t() if layout == grass.DY_MxT else dY
    want = rho.double()[:, None] * (rows.double()[:, idx.long()].t() @ X.double())
    for slices in (1, 2, 7):
        grass.set_test_option(grass.TEST_MAX_K_SLICES, slices)
        assert grass.cgrad_plan(T, n, r, grass.BF16, layout)[0] == 256
        ws = grass.workspace(grass.cgrad_workspace(T, m, n, r, grass.BF16, layout))
        results = []
        for tile, kernel in ((128, grass.KERNEL_128), (192, grass.KERNEL_128_256),
                             (256, grass.KERNEL_256_ROWS if layout == grass.DY_MxT and T % 32 == 0 else grass.KERNEL_256)):
            grass.set_test_option(grass.TEST_RUN_TILE, tile)
            GC = torch.full((r, n), float("nan"), device=DEV)
            grass.compressed_grad(dY, X, idx, rho, GC, ws, layout)
            assert grass.last_kernel() == kernel
            results.append(GC)
        # products of bf16 values are exact in fp32; their sum is off by about sqrt(T) * 2^-24, 3e-6 here
        assert float((results[0].double() - want).norm() / want.norm()) <= 1e-5
        assert torch.equal(results[0], results[1]) and torch.equal(results[0], results[2])
