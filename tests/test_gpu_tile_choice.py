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
