"""GPU parity of the 128 x 256 tile at the edges of its tiles, its ring (three K tiles of 32) and its
K slices, gathered and dense, against the fp64 oracle.  Bound as for the other bf16 kernels: products
exact in fp32, sums of T of them off by about sqrt(T) * 2^-24; TOL_F32 covers it."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_2406_17660_amd import grass
from gpu_util import DEV, TOL_F32, rel_fro, to_f64, to_np

pytestmark = pytest.mark.gpu


def _run(T, m, n, r, slices=0, seed=0, tile=192):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    # Inf behind the last token and behind the last column: must not be multiplied in
    flat = torch.full((T + 40, n + 8), float("inf"), dtype=torch.bfloat16, device=DEV)
    X = flat[:T, :n]
    X.copy_(torch.randn(T, n, generator=gen, device=DEV))
    dY = torch.randn(T, m, generator=gen, device=DEV).to(torch.bfloat16)
    idx = torch.randint(0, m, (r,), generator=gen, device=DEV).sort()[0].to(torch.int32)
    rho = torch.rand(r, generator=gen, device=DEV) + 0.5
    grass.set_test_option(grass.TEST_GEMM_TILE, tile)
    grass.set_test_option(grass.TEST_MAX_K_SLICES, slices)
    GC = torch.full((r, n), float("nan"), device=DEV)
    grass.compressed_grad(dY, X, idx, rho, GC, grass.workspace(grass.cgrad_workspace(T, m, n, r, grass.BF16)))
    assert rel_fro(to_np(GC), ref.compressed_grad(to_f64(dY), to_f64(X), to_np(idx), to_np(rho))) <= TOL_F32
    G = torch.full((m, n), float("nan"), device=DEV)
    grass.dense_grad(dY, X, G, grass.workspace(grass.dense_workspace(T, m, n, grass.BF16)))
    assert rel_fro(to_np(G), to_f64(dY).T @ to_f64(X)) <= TOL_F32


@pytest.mark.parametrize("T", [32, 33, 64, 95, 96, 97, 128, 160, 192, 200, 224, 256, 1001])
@pytest.mark.parametrize("m,n,r", [(8, 8, 1), (128, 256, 127), (136, 264, 130), (264, 520, 257)])
def test_tiles_and_ring(T, m, n, r):
    _run(T, m, n, r)


@pytest.mark.parametrize("slices", [1, 2, 5, 9, 40])
def test_slices_end_in_a_ragged_tile(slices):
    _run(2477, 304, 520, 260, slices)


@pytest.mark.parametrize("T", [32, 33, 64, 95, 96, 97, 128, 193, 1001])
@pytest.mark.parametrize("m,n,r", [(8, 8, 1), (128, 128, 127), (136, 136, 130), (264, 392, 257)])
def test_128_columns(T, m, n, r):
    _run(T, m, n, r, tile=128)
    _run(T, m, n, r, 1, tile=128)


@pytest.mark.parametrize("slices", [2, 5, 40])
def test_128_columns_slices_end_in_a_ragged_tile(slices):
    _run(2477, 304, 520, 260, slices, tile=128)
