"""A call writes nothing outside the workspace its query asked for: the bytes behind it (and before
it) keep their pattern."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_2406_17660_amd import grass
from gpu_util import DEV, rel_fro, to_f64, to_np
from test_gpu_parity import make_idx, randn, run_step_cols, run_step_group

pytestmark = pytest.mark.gpu
BF = torch.bfloat16
GUARD = 1 << 20


def guarded(nbytes, shift=0):
    """(workspace of nbytes that starts `shift` bytes after a 256-byte boundary, guard check)."""
    buf = torch.full((GUARD + nbytes + shift + GUARD,), 0x5A, dtype=torch.uint8, device=DEV)
    lo, hi = GUARD + shift, GUARD + shift + nbytes

    def untouched():
        return bool((buf[:lo] == 0x5A).all()) and bool((buf[hi:] == 0x5A).all())
    return buf[lo:hi], untouched


@pytest.mark.parametrize("shift", [0, 252])
@pytest.mark.parametrize("T,n,m,rs", [
    (480, 256, 512, (64,) * 4), (1024, 64, 512, (32,) * 8), (2048, 256, 512, (32,) * 8),
    (8192, 512, 512, (32,) * 8), (2048, 264, 384, (9, 17, 33, 64, 65, 127, 128, 1))])
def test_narrow_groups_stay_inside_the_queried_workspace(T, n, m, rs, shift):
    X = randn((T, n), BF, 1)
    dYs = [randn((T, m), BF, 2 + i, scale=0.1) for i in range(len(rs))]
    host = [make_idx(m, r, 20 + i, duplicates=False) for i, r in enumerate(rs)]
    idxs = [torch.from_numpy(i).to(DEV) for i, _ in host]
    rhos = [torch.from_numpy(p).to(DEV) for _, p in host]
    want = [ref.compressed_grad(to_np(dY), to_np(X), i, p) for dY, (i, p) in zip(dYs, host)]
    total = sum((r + 7) // 8 * 8 for r in rs)
    assert grass.cgrad_plan(T, n, total, grass.BF16, m=m, count=len(rs))[0] == 0

    GCs = [torch.full((r, n), float("nan"), device=DEV) for r in rs]
    ws, untouched = guarded(grass.cgrad_group_workspace(T, n, rs, grass.BF16), shift)
    grass.compressed_grad_group(dYs, X, idxs, rhos, GCs, ws)
    assert untouched()
    for got, w in zip(GCs, want):
        assert np.isfinite(to_np(got)).all() and rel_fro(to_f64(got), w) <= 2e-5

    Ms, Vs = ([torch.zeros((r, n), device=DEV) for r in rs] for _ in range(2))
    Ws = [torch.zeros((m, n), dtype=BF, device=DEV) for _ in rs]
    ws, untouched = guarded(grass.step_group_workspace(T, n, rs, grass.BF16), shift)
    grass.step_group(dYs, X, idxs, rhos, Ms, Vs, Ws, 1e-3, 0.9, 0.999, 1e-8, 1, 0.5, ws)
    assert untouched()
    for M, w in zip(Ms, want):
        assert rel_fro(to_f64(M), 0.1 * w) <= 2e-5


@pytest.mark.parametrize("shift", [0, 255])
@pytest.mark.parametrize("T,m,n", [(16071, 216, 507), (4096, 248, 255), (513, 127, 131)])
def test_row_statistic_stays_inside_the_queried_workspace(T, m, n, shift):
    """G and the product's partial tiles one after the other, from a start that is not aligned and
    with an m x n whose bytes are not a multiple of 256."""
    X, dY = randn((T, n), BF, 5), randn((T, m), BF, 6, scale=0.1)
    ss = torch.full((m,), float("nan"), device=DEV)
    ws, untouched = guarded(grass.grad_row_stats_workspace(T, m, n, grass.BF16, grass.DY_TxM, m, n), shift)
    grass.grad_row_stats(dY, X, ss, ws)
    assert untouched()
    # squares of sums that are off by about sqrt(T) * 2^-24 each: twice that
    assert rel_fro(to_np(ss), ref.row_stats(ref.full_grad(to_np(dY), to_np(X)))) <= 2e-5


@pytest.mark.parametrize("room", ["least", "half", "query"])
@pytest.mark.parametrize("T,m,n", [(8192, 200, 96), (2047, 259, 261)])
def test_row_statistic_of_fp32_inputs_takes_a_short_workspace(T, m, n, room):
    """Room for G alone is enough: the partial tiles of the product are an aid."""
    X, dY = randn((T, n), torch.float32, 7), randn((T, m), torch.float32, 8, scale=0.1)
    least = m * n * 4 + 256
    query = grass.grad_row_stats_workspace(T, m, n, grass.F32)
    assert least < query
    ss = torch.full((m,), float("nan"), device=DEV)
    ws, untouched = guarded({"least": least, "half": (least + query) // 2, "query": query}[room], 0)
    grass.grad_row_stats(dY, X, ss, ws)
    assert untouched()
    assert rel_fro(to_np(ss), ref.row_stats(ref.full_grad(to_np(dY), to_np(X)))) <= 2e-5
    with pytest.raises(grass.GrassError):
        grass.grad_row_stats(dY, X, ss, guarded(least - 1)[0])


@pytest.mark.parametrize("T,m,n,r", [(6672, 40, 1394, 5), (2513, 300, 257, 130), (4096, 128, 128, 128), (1500, 64, 1030, 9)])
def test_fp32_results_do_not_depend_on_room_beyond_the_query(T, m, n, r):
    """A workspace of the queried size gives the slices that an unlimited one gives: the same bits."""
    X, dY = randn((T, n), torch.float32, 9), randn((T, m), torch.float32, 10)
    idx, rho = (torch.from_numpy(a).to(DEV) for a in make_idx(m, r, 11, False))
    need = grass.cgrad_workspace(T, m, n, r, grass.F32)
    outs = []
    for nbytes in (need, 4 * need):
        GC = torch.full((r, n), float("nan"), device=DEV)
        ws, untouched = guarded(nbytes)
        grass.compressed_grad(dY, X, idx, rho, GC, ws)
        assert untouched()
        outs.append(GC)
    assert torch.equal(*outs)


def rounded(nbytes):
    return (nbytes + 255) // 256 * 256


@pytest.mark.parametrize("T,n,ms,rs,want_gc", [
    (2048, 256, (256,), (16,), False), (1500, 50, (70, 64, 9), (33, 64, 1), True),
    (512, 260, (40, 64), (40, 0), False)])
def test_fp32_step_with_room_for_the_gradient_alone(monkeypatch, T, n, ms, rs, want_gc):
    """Not one slice of partial tiles fits: the product is stored directly, Adam and the row update
    follow as a kernel of their own.  Duplicate rows, an empty set."""
    least = 256 + sum(rounded(4 * r * n) for r in rs)
    assert least < grass.step_group_workspace(T, n, rs, grass.F32)
    monkeypatch.setattr(grass, "step_group_workspace", lambda *a: least)
    run_step_group(torch.float32, torch.float32, torch.float32, T, n, ms, rs, want_gc, None)
    monkeypatch.setattr(grass, "step_group_workspace", lambda *a: least - 1)
    with pytest.raises(grass.GrassError):
        run_step_group(torch.float32, torch.float32, torch.float32, T, n, ms, rs, want_gc, None)


@pytest.mark.parametrize("T,m,n,r,want_gc", [(2048, 256, 64, 16, False), (300, 130, 50, 17, True)])
def test_fp32_column_step_with_room_for_the_gradient_alone(monkeypatch, T, m, n, r, want_gc):
    least = 256 + rounded(4 * r * m)
    assert least < grass.step_cols_workspace(T, m, n, r, grass.F32)
    monkeypatch.setattr(grass, "step_cols_workspace", lambda *a: least)
    run_step_cols(torch.float32, torch.float32, T, m, n, r, True, want_gc, None)


@pytest.mark.parametrize("T", [512, 1000, 1536])
def test_fp32_step_and_separate_call_differ_in_summation_order_alone(T):
    """Below 1024 tokens a step splits K where the separate call does not: equal within the rounding
    of their sums (sqrt(T) * 2^-24 each), and bit for bit with one slice in both."""
    m, n, r = 256, 256, 16
    X, dY = randn((T, n), torch.float32, 12), randn((T, m), torch.float32, 13, scale=0.1)
    idx, rho = (torch.from_numpy(a).to(DEV) for a in make_idx(m, r, 14, False))

    def both():
        outs = [torch.full((r, n), float("nan"), device=DEV) for _ in range(2)]
        grass.compressed_grad(dY, X, idx, rho, outs[0],
                              grass.workspace(max(grass.cgrad_workspace(T, m, n, r, grass.F32), 16)))
        M, V, W = (torch.zeros((k, n), device=DEV) for k in (r, r, m))
        grass.step_group([dY], X, [idx], [rho], [M], [V], [W], 1e-3, 0.9, 0.999, 1e-8, 1, 0.5,
                         grass.workspace(grass.step_group_workspace(T, n, [r], grass.F32)), GCs=[outs[1]])
        return outs
    call, step = both()
    assert rel_fro(to_f64(step), to_f64(call)) <= 4 * T ** 0.5 * 2.0 ** -24
    grass.set_test_option(grass.TEST_MAX_K_SLICES, 1)
    assert torch.equal(*both())
