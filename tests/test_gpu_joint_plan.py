"""Tile and K slices chosen together (products of up to 8192 tokens): random layers on both sides of the choice, in
both layouts, odd widths and columns, against 64-bit products, with the workspace the query asks for and with the least
one that a call accepts.  The workspace holds NaN before each call, so a slice that nobody writes shows.  Bound: products
of bf16 values are exact in fp32, sums of T of them off by about sqrt(T) * 2^-24 = 5e-6; TOL_F32 (1e-5) covers it."""
import random

import pytest
import torch

from paper_2406_17660_amd import grass
from gpu_util import DEV, TOL_F32

pytestmark = pytest.mark.gpu
BF = torch.bfloat16


def _rel(got, want):
    return float((got.double() - want).norm() / want.norm())


def _case(seed):
    rng = random.Random(seed)
    T = rng.choice([32, 63, 257, 640, 1001, 2080, 4099, 8192, 8193])
    m, n = (rng.choice([8, 128, 261, 488, 1030, 2376]) + 8 * rng.randrange(4) for _ in range(2))
    return T, m, n, max(1, m // rng.choice([1, 4, 8])), rng.choice([grass.DY_TxM, grass.DY_MxT])


@pytest.mark.parametrize("seed", range(60))
def test_products_and_steps(seed):
    T, m, n, r, layout = _case(seed)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    dY = torch.randn((T, m) if layout == grass.DY_TxM else (m, T), generator=gen, device=DEV).to(BF)
    X = torch.randn(T, n, generator=gen, device=DEV).to(BF)
    W = torch.randn(m, n, generator=gen, device=DEV).to(BF)
    idx = torch.randperm(m, generator=gen, device=DEV)[:r].sort()[0].to(torch.int32)
    rho = torch.rand(r, generator=gen, device=DEV) + 0.5
    full = (dY.double().t() if layout == grass.DY_TxM else dY.double()) @ X.double()
    want = rho.double()[:, None] * full[idx.long()]

    c = min(r, n)  # columns of W: the transposed problem
    cols = torch.randperm(n, generator=gen, device=DEV)[:c].sort()[0].to(torch.int32)
    want_cols = rho.double()[:c, None] * full.t()[cols.long()]

    def check(nbytes_cgrad, nbytes_dense, nbytes_step, nbytes_cols):
        GC, G = torch.full((r, n), float("nan"), device=DEV), torch.full((m, n), float("nan"), device=DEV)
        grass.compressed_grad(dY, X, idx, rho, GC, grass.workspace(nbytes_cgrad).fill_(255), layout)
        assert _rel(GC, want) <= TOL_F32
        grass.dense_grad(dY, X, G, grass.workspace(nbytes_dense).fill_(255), layout)
        assert _rel(G, full) <= TOL_F32
        M, V = torch.zeros(r, n, device=DEV), torch.zeros(r, n, device=DEV)
        grass.step_group([dY], X, [idx], [rho], [M], [V], [W], 1e-3, 0.9, 0.999, 1e-8, 1, 0.25,
                         grass.workspace(nbytes_step).fill_(255), layout=layout)
        assert _rel(M, 0.1 * want) <= TOL_F32
        if layout == grass.DY_TxM:
            M, V, U = (torch.zeros(c, m, device=DEV) for _ in range(3))
            grass.step_cols(dY, X, cols, rho[:c], M, V, U, W, 1e-3, 0.9, 0.999, 1e-8, 1, 0.25,
                            grass.workspace(nbytes_cols).fill_(255))
            assert _rel(M, 0.1 * want_cols) <= TOL_F32

    query = (grass.cgrad_workspace(T, m, n, r, grass.BF16, layout), grass.dense_workspace(T, m, n, grass.BF16, layout),
             grass.step_group_workspace(T, n, [r], grass.BF16, layout), grass.step_cols_workspace(T, m, n, c, grass.BF16))
    least = (grass.least_workspace(grass.CALL_CGRAD, T, n, [r], layout), grass.least_workspace(grass.CALL_DENSE, T, n, [m], layout),
             grass.least_workspace(grass.CALL_STEP, T, n, [r], layout), grass.least_workspace(grass.CALL_STEP, T, m, [c]))
    assert all(a <= b for a, b in zip(least, query))
    check(*query)
    check(*least)


@pytest.mark.parametrize("layout", [grass.DY_TxM, grass.DY_MxT])
@pytest.mark.parametrize("T,m,n,rs", [(257, 1030, 264, (60, 9)), (640, 600, 1032, (128, 40, 40)), (1001, 261, 517, (30, 31)),
                                      (2080, 1024, 600, (256, 256)), (8192, 544, 264, (50, 7, 120))])
def test_sets_in_one_panel(T, m, n, rs, layout):
    """Several sets that share X in one step, with the workspace of the query and with the least one."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(T)
    dYs = [torch.randn((T, m) if layout == grass.DY_TxM else (m, T), generator=gen, device=DEV).to(BF) for _ in rs]
    X = torch.randn(T, n, generator=gen, device=DEV).to(BF)
    idxs = [torch.randperm(m, generator=gen, device=DEV)[:r].sort()[0].to(torch.int32) for r in rs]
    rhos = [torch.rand(r, generator=gen, device=DEV) + 0.5 for r in rs]
    for nbytes in (grass.step_group_workspace(T, n, rs, grass.BF16, layout), grass.least_workspace(grass.CALL_STEP, T, n, rs, layout)):
        Ms, Vs = ([torch.zeros(r, n, device=DEV) for r in rs] for _ in range(2))
        Ws = [torch.zeros(m, n, dtype=BF, device=DEV) for _ in rs]
        grass.step_group(dYs, X, idxs, rhos, Ms, Vs, Ws, 1e-3, 0.9, 0.999, 1e-8, 1, 0.25, grass.workspace(nbytes).fill_(255), layout=layout)
        for dY, idx, rho, M in zip(dYs, idxs, rhos, Ms):
            d = dY.double() if layout == grass.DY_TxM else dY.double().t()
            assert _rel(M, 0.1 * rho.double()[:, None] * (d[:, idx.long()].t().contiguous() @ X.double())) <= TOL_F32


def test_slices_of_a_short_product_and_of_a_long_one():
    grass.set_test_option(grass.TEST_MAX_K_SLICES, 128)
    alone = grass.cgrad_plan(4270, 488, 166, grass.BF16)
    long = grass.cgrad_plan(65536, 2048, 512, grass.BF16)
    grass.set_test_option(grass.TEST_MAX_K_SLICES, 0)
    assert grass.cgrad_plan(4270, 488, 166, grass.BF16)[1] > alone[1]
    assert grass.cgrad_plan(65536, 2048, 512, grass.BF16) == long


@pytest.mark.parametrize("T", [256, 272, 1280, 8192, 32768, 32784])
@pytest.mark.parametrize("m,n,r,count", [(512, 512, 128, 1), (264, 200, 40, 3), (512, 264, 7, 1)])
def test_slices_of_narrow_layers(T, m, n, r, count):
    """The gather inside the product, alone and grouped: slices for the workspace of the query, and for the least one
    that is accepted, into which fewer of them fit where it is the smaller one by a slice or more."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(T)
    dYs = [torch.randn(T, m, generator=gen, device=DEV).to(BF) for _ in range(count)]
    X = torch.randn(T, n, generator=gen, device=DEV).to(BF)
    idx = torch.randperm(m, generator=gen, device=DEV)[:r].sort()[0].to(torch.int32)
    rho = torch.rand(r, generator=gen, device=DEV) + 0.5
    query = grass.step_group_workspace(T, n, [r] * count, grass.BF16)
    least = grass.least_workspace(grass.CALL_STEP, T, n, [r] * count)
    rows = (r + 7) // 8 * 8 * count
    tile, slices = grass.cgrad_plan(T, n, rows if count > 1 else r, grass.BF16, m=m, count=count)
    slice_bytes = rows * ((n + 255) // 256 * 256) * 4
    assert tile == 0 and least <= query

    def step(nbytes):
        Ms, Vs = ([torch.zeros(r, n, device=DEV) for _ in range(count)] for _ in range(2))
        Ws = [torch.zeros(m, n, dtype=BF, device=DEV) for _ in range(count)]
        ws = grass.workspace(nbytes).fill_(255)
        grass.step_group(dYs, X, [idx] * count, [rho] * count, Ms, Vs, Ws, 1e-3, 0.9, 0.999, 1e-8, 1, 0.25, ws)
        assert grass.last_kernel() == grass.KERNEL_NARROW
        for dY, M in zip(dYs, Ms):
            want = 0.1 * rho.double()[:, None] * (dY.double()[:, idx.long()].t().contiguous() @ X.double())
            assert _rel(M, want) <= TOL_F32
        return -(-(int((ws != 255).nonzero().max()) + 1) // slice_bytes)  # the slices that were written

    assert step(query) == slices
    room = (least - 256 - 256 - sum((r * n * 4 + 255) // 256 * 256 for _ in range(count))) // slice_bytes
    used = step(least)
    assert used <= room and (used < slices or slices <= room)
    with pytest.raises(grass.GrassError) as e:
        step(least - 256)
    assert e.value.code == grass.ERR_WORKSPACE


def test_least_workspace_holds_fewer_slices_of_a_narrow_layer():
    """(so that the above runs a plan that the room bounds)"""
    least = grass.least_workspace(grass.CALL_CGRAD, 1280, 512, [128])
    assert grass.cgrad_plan(1280, 512, 128, grass.BF16, m=512)[1] * 128 * 512 * 4 > least


@pytest.mark.parametrize("T,m,n", [(192, 40, 3522), (192, 24, 1851), (960, 16, 1227), (536, 232, 702), (1001, 520, 264), (640, 264, 1030)])
@pytest.mark.parametrize("a_off,x_off", [(0, 0), (1, 0), (0, 1), (1, 1)])
def test_a_workspace_beyond_the_query_changes_no_sum(T, m, n, a_off, x_off):
    """The query holds the plan that is taken with any amount of room, wherever the operands lie: the sums are the same."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(T)

    def operand(width, off):
        return torch.randn(T * width + 8, generator=gen, device=DEV).to(BF)[off:off + T * width].view(T, width)

    dY, X = operand(m, a_off), operand(n, x_off)
    query = grass.dense_workspace(T, m, n, grass.BF16)
    G, H = torch.empty(m, n, device=DEV), torch.empty(m, n, device=DEV)
    grass.dense_grad(dY, X, G, grass.workspace(query))
    grass.dense_grad(dY, X, H, grass.workspace(4 * query))
    assert torch.equal(G, H)
    assert _rel(G, dY.double().t() @ X.double()) <= TOL_F32


@pytest.mark.parametrize("T,m,n", [(256, 256, 256), (467, 3128, 2736), (128, 720, 128), (384, 2704, 3024)])
def test_full_gradients_of_one_planned_slice_stay_in_one(T, m, n):
    """The product of one slice stores a full gradient itself, which saves more than slices would: nothing is written to
    the workspace."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(T)
    dY, X = (torch.randn(T, w, generator=gen, device=DEV).to(BF) for w in (m, n))
    G = torch.full((m, n), float("nan"), device=DEV)
    ws = grass.workspace(grass.dense_workspace(T, m, n, grass.BF16)).fill_(165)
    grass.dense_grad(dY, X, G, ws)
    assert bool((ws == 165).all())
    assert _rel(G, dY.double().t() @ X.double()) <= TOL_F32
