"""GPU parity of the bf16 products on operands in any position (odd widths, sliced tensors, bases off
16 bytes) and with any number of tokens, against the fp64 oracle.

Everything around the operands holds Inf: a value read from outside a row, or a token past the end
that is not cleared, turns an output into Inf or NaN.  Bound: products of bf16 values are exact
in fp32, a sum of T of them is off by about sqrt(T) * 2^-24 relatively, 3e-6 at the largest T
here; TOL_F32 (1e-5) covers it."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_2406_17660_amd import grass
from gpu_util import DEV, TOL_F32, rel_fro, to_f64, to_np

pytestmark = pytest.mark.gpu
BF = torch.bfloat16


def _framed(rows, cols, ld, first, gen):
    """A rows x cols bf16 matrix with leading dimension ld that starts `first` elements into a buffer
    of Inf (16-byte aligned when first is 8)."""
    flat = torch.full((first + rows * ld + 64,), float("inf"), dtype=BF, device=DEV)
    view = flat[first:first + rows * ld].view(rows, ld)[:, :cols]
    view.copy_(torch.randn(rows, cols, generator=gen, device=DEV))
    return view


def _check(T, m, n, r, layout, ldy_pad, ldx_pad, first, seed=0, kernel=None):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    X = _framed(T, n, n + ldx_pad, first, gen)
    dY = _framed(m, T, T + ldy_pad, first, gen) if layout == grass.DY_MxT else \
        _framed(T, m, m + ldy_pad, first, gen)
    idx = torch.randint(0, m, (r,), generator=gen, device=DEV).sort()[0].to(torch.int32)
    rho = torch.rand(r, generator=gen, device=DEV) + 0.5
    d = to_f64(dY)
    d = np.ascontiguousarray(d.T) if layout == grass.DY_MxT else d
    want = ref.compressed_grad(d, to_f64(X), to_np(idx), to_np(rho))
    GC = torch.full((r, n), float("nan"), device=DEV)
    grass.compressed_grad(dY, X, idx, rho, GC,
                          grass.workspace(grass.cgrad_workspace(T, m, n, r, grass.BF16, layout)), layout)
    assert kernel is None or grass.last_kernel() == kernel
    assert rel_fro(to_np(GC), want) <= TOL_F32
    G = torch.full((m, n), float("nan"), device=DEV)
    grass.dense_grad(dY, X, G, grass.workspace(grass.dense_workspace(T, m, n, grass.BF16, layout)), layout)
    assert rel_fro(to_np(G), d.T @ to_f64(X)) <= TOL_F32


# tokens around the K tiles of both kernels (32 and 64) and around the six whole tiles from which the
# large tile's steady loop runs; widths around a chunk (8), a wavefront's block (128) and a tile
@pytest.mark.parametrize("tile", [128, 256])
@pytest.mark.parametrize("T", [1, 31, 32, 33, 63, 64, 95, 129, 192, 200, 257, 1000])
@pytest.mark.parametrize("m,n,first,pad", [(9, 9, 8, 0), (257, 135, 9, 0), (263, 250, 8, 3), (120, 391, 15, 2)])
def test_any_position(tile, T, m, n, first, pad):
    grass.set_test_option(grass.TEST_GEMM_TILE, tile)
    _check(T, m, n, min(m, 140), grass.DY_TxM, pad, pad, first)


# the same on the large tile's kernel for both operands in any position (X on a 2-byte boundary, which no copy reads),
# on slices of 64 tokens
@pytest.mark.parametrize("slices", [1, 3])
@pytest.mark.parametrize("T", [32, 33, 63, 64, 95, 129, 192, 200, 257, 1000])
@pytest.mark.parametrize("m,n,first,pad", [(9, 9, 9, 0), (257, 135, 9, 0), (263, 250, 11, 3), (120, 391, 15, 2)])
def test_any_position_on_the_large_tile(T, m, n, first, pad, slices):
    grass.set_test_option(grass.TEST_RUN_TILE, 256)
    grass.set_test_option(grass.TEST_MAX_K_SLICES, slices)
    _check(T, m, n, min(m, 140), grass.DY_TxM, pad, pad, first, kernel=grass.KERNEL_256_UNALIGNED)
    assert grass.last_kernel() == grass.KERNEL_256_UNALIGNED  # the full gradient too


@pytest.mark.parametrize("tile", [128, 256])
@pytest.mark.parametrize("T", [33, 64, 320, 2501])
@pytest.mark.parametrize("m,n", [(264, 248), (3, 5), (256, 7), (6, 256)])
def test_ragged_tokens_of_aligned_and_tiny_operands(tile, T, m, n):
    grass.set_test_option(grass.TEST_GEMM_TILE, tile)
    _check(T, m, n, min(m, 136), grass.DY_TxM, -m % 8, -n % 8, 8)


@pytest.mark.parametrize("T,n,first", [(320, 261, 8), (321, 261, 8), (320, 264, 9), (45, 300, 11)])
def test_mxt_storage(T, n, first):
    grass.set_test_option(grass.TEST_GEMM_TILE, 256)
    _check(T, 270, n, 260, grass.DY_MxT, -T % 8, 0, first)


@pytest.mark.parametrize("slices", [1, 3, 5])
def test_slices_end_in_a_ragged_tile(slices):
    grass.set_test_option(grass.TEST_GEMM_TILE, 256)
    grass.set_test_option(grass.TEST_MAX_K_SLICES, slices)
    _check(2477, 300, 515, 260, grass.DY_TxM, 0, 0, 8)
    _check(2477, 304, 520, 260, grass.DY_TxM, 0, 0, 8)


@pytest.mark.parametrize("T,m,n", [(96, 5000, 2051), (96, 2051, 5000)])
def test_full_gradient_whose_odd_operand_is_copied(T, m, n):
    _check(T, m, n, 8, grass.DY_TxM, 0, 0, 8)


# Aligned left operand, X in any position: every length of the ring's start (nine whole tiles), of its steady loop
# (four tiles a turn) and of its end, one and two row and column tiles, a last slice of one to nine tiles.  X starts on
# a 2-byte boundary, which no copy reads.
def _left_operand_by_load_to_lds(T, r, n, slices):
    grass.set_test_option(grass.TEST_RUN_TILE, 256)
    grass.set_test_option(grass.TEST_UNALIGNED_X, 1)
    grass.set_test_option(grass.TEST_MAX_K_SLICES, slices)
    _check(T, 264, n, r, grass.DY_TxM, 0, 0, 9, kernel=grass.KERNEL_256_UNALIGNED_X)


@pytest.mark.parametrize("rest", [0, 5])
@pytest.mark.parametrize("tiles", [*range(1, 19), 21, 22])
def test_left_operand_by_load_to_lds(tiles, rest):
    _left_operand_by_load_to_lds(32 * tiles + rest, 140, 261, 1)
    _left_operand_by_load_to_lds(32 * tiles + rest, 262, 250, 1)


@pytest.mark.parametrize("last", range(1, 10))
def test_left_operand_by_load_to_lds_in_slices(last):
    """Slices of 20 K tiles (10 of the plan's 64 tokens) and a shorter one."""
    T = 32 * (20 * 19 + last) - (3 if last % 2 else 0)
    grass.set_test_option(grass.TEST_MAX_K_SLICES, 20)
    assert grass.cgrad_plan(T, 261, 260, grass.BF16) in ((128, 20), (256, 20))
    _left_operand_by_load_to_lds(T, 260, 261, 20)


def test_left_operand_by_load_to_lds_is_chosen():
    """Odd width, more than one row tile and 64 K tiles per slice."""
    dY, X = torch.zeros(65536, 512, dtype=BF, device=DEV), torch.zeros(65536, 2045, dtype=BF, device=DEV)
    G = torch.empty(512, 2045, device=DEV)
    grass.dense_grad(dY, X, G, grass.workspace(grass.dense_workspace(65536, 512, 2045, grass.BF16)))
    assert grass.last_kernel() == grass.KERNEL_256_UNALIGNED_X


# The operands' ways exchanged: X in aligned chunks, dY of a full gradient in any position.
def _x_by_load_to_lds(T, m, n, slices):
    grass.set_test_option(grass.TEST_RUN_TILE, 256)
    grass.set_test_option(grass.TEST_UNALIGNED_X, 1)
    grass.set_test_option(grass.TEST_MAX_K_SLICES, slices)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(T)
    dY, X = _framed(T, m, m, 9, gen), _framed(T, n, n + 8, 8, gen)
    G = torch.full((m, n), float("nan"), device=DEV)
    grass.dense_grad(dY, X, G, grass.workspace(grass.dense_workspace(T, m, n, grass.BF16)))
    assert grass.last_kernel() == grass.KERNEL_256_UNALIGNED_DY
    assert rel_fro(to_np(G), to_f64(dY).T @ to_f64(X)) <= TOL_F32


@pytest.mark.parametrize("rest", [0, 5])
@pytest.mark.parametrize("tiles", [*range(1, 19), 21, 22])
def test_x_by_load_to_lds(tiles, rest):
    _x_by_load_to_lds(32 * tiles + rest, 261, 136, 1)
    _x_by_load_to_lds(32 * tiles + rest, 141, 264, 1)


@pytest.mark.parametrize("last", range(1, 10))
def test_x_by_load_to_lds_in_slices(last):
    _x_by_load_to_lds(32 * (20 * 19 + last) - (3 if last % 2 else 0), 261, 264, 20)


def test_x_by_load_to_lds_is_chosen():
    dY, X = torch.zeros(65536, 2045, dtype=BF, device=DEV), torch.zeros(65536, 512, dtype=BF, device=DEV)
    G = torch.empty(2045, 512, device=DEV)
    grass.dense_grad(dY, X, G, grass.workspace(grass.dense_workspace(65536, 2045, 512, grass.BF16)))
    assert grass.last_kernel() == grass.KERNEL_256_UNALIGNED_DY


# A full gradient of one slice is stored by the product itself (by the staged 128 tile through partial tiles): edges of
# every tile, an output with padded rows, whose padding stays as it is.
@pytest.mark.parametrize("tile", [128, 192, 256])
@pytest.mark.parametrize("T", [32, 333])
@pytest.mark.parametrize("m,n", [(8, 8), (128, 256), (136, 264), (264, 248), (512, 128), (257, 264), (264, 261), (131, 517)])
def test_full_gradient_of_one_slice(tile, T, m, n):
    grass.set_test_option(grass.TEST_RUN_TILE, tile)
    grass.set_test_option(grass.TEST_MAX_K_SLICES, 1)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(T)
    dY, X = _framed(T, m, m, 9 if m % 8 else 8, gen), _framed(T, n, n, 9 if n % 8 else 8, gen)
    out = torch.full((m + 1, n + 3), 7.0, device=DEV)
    G = out[:m, :n]
    ws = grass.workspace(grass.dense_workspace(T, m, n, grass.BF16)).fill_(165)
    grass.dense_grad(dY, X, G, ws)
    assert rel_fro(to_np(G), to_f64(dY).T @ to_f64(X)) <= TOL_F32
    assert bool((out[m] == 7).all()) and bool((out[:m, n:] == 7).all())
    if m % 8 == 0 and n % 8 == 0:  # nothing is copied ahead of the product: a workspace as it was shows that G went past it
        assert grass.last_kernel() != grass.KERNEL_128_STAGED and bool((ws == 165).all())
    elif grass.last_kernel() == grass.KERNEL_128_STAGED:  # (stores partial tiles)
        assert tile != 256 and not bool((ws == 165).all())


@pytest.mark.parametrize("over", ["dY", "X"])
@pytest.mark.parametrize("tile", [128, 192, 256])
@pytest.mark.parametrize("m,n", [(512, 512), (520, 264), (257, 264), (264, 261)])
def test_full_gradient_over_an_input(over, tile, m, n):
    """G may lie over a bf16 input: no workgroup stores while another still reads (dY and X have room for it)."""
    T = 2048
    grass.set_test_option(grass.TEST_RUN_TILE, tile)
    grass.set_test_option(grass.TEST_MAX_K_SLICES, 1)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(m)
    dY, X = (torch.randn(T, w, generator=gen, device=DEV).to(BF) for w in (m, n))
    want = to_f64(dY).T @ to_f64(X)
    under = dY if over == "dY" else X
    G = under.view(-1)[:2 * m * n].view(torch.float32).view(m, n)
    grass.dense_grad(dY, X, G, grass.workspace(grass.dense_workspace(T, m, n, grass.BF16)))
    assert G.data_ptr() == under.data_ptr() and rel_fro(to_np(G), want) <= TOL_F32
