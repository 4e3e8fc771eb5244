"""The fused tail of a step (sum over the K slices, Adam, row or column update in one kernel) where rows
are not 16-byte aligned, against the same step in separate calls: compressed_grad, then adam_scatter,
or adam_rows and scatter_update_cols, each of which is checked against the oracle elsewhere.

Both routes add the slices in the same order and use the same arithmetic per element, so every
output is compared bit for bit."""
import pytest
import torch

from paper_2406_17660_amd import grass
from gpu_util import DEV

pytestmark = pytest.mark.gpu
ADAM = (1e-2, 0.9, 0.999, 1e-8, 3)


def _setup(T, m, n, r, dtype, sdt, wdt, wpad, repeat):
    g = torch.Generator(device=DEV).manual_seed(T + n + r)
    dY = torch.randn(T, m, generator=g, device=DEV).to(dtype)
    X = torch.randn(T, n, generator=g, device=DEV).to(dtype)
    idx = torch.randint(0, max(1, r // 3), (r,), generator=g, device=DEV) if repeat else \
        torch.randperm(m, generator=g, device=DEV)[:r]
    idx = idx.sort()[0].to(torch.int32)
    rho = torch.rand(r, generator=g, device=DEV) + 0.5
    M = torch.randn(r, n, generator=g, device=DEV).to(sdt)
    V = torch.rand(r, n, generator=g, device=DEV).to(sdt)
    W = torch.randn(m, n + wpad, generator=g, device=DEV).to(wdt)[:, :n]
    return dY, X, idx, rho, M, V, W


def _same(got, want):
    for name in want:
        assert torch.equal(got[name], want[name]), name


# n around a wavefront, a workgroup's 256 and its 1024 columns; aligned rows with an odd leading dimension
# of W; 1 to 8 slices are added in order, more by four wavefronts
@pytest.mark.parametrize("n,wpad", [(1, 0), (63, 2), (257, 0), (1023, 0), (1025, 0), (512, 1), (2051, 3)])
@pytest.mark.parametrize("slices", [1, 2, 8, 9, 40])
@pytest.mark.parametrize("sdt,wdt,repeat,keep", [
    (torch.float32, torch.bfloat16, False, True), (torch.bfloat16, torch.bfloat16, True, False),
    (torch.float32, torch.float32, True, True), (torch.bfloat16, torch.float32, False, False)])
def test_rows(n, wpad, slices, sdt, wdt, repeat, keep):
    T, m, r = 2592, 140, 37
    grass.set_test_option(grass.TEST_MAX_K_SLICES, slices)
    dY, X, idx, rho, M, V, W = _setup(T, m, n, r, torch.bfloat16, sdt, wdt, wpad, repeat)
    lr, b1, b2, eps, t = ADAM
    GC = torch.empty(r, n, device=DEV)
    grass.compressed_grad(dY, X, idx, rho, GC, grass.workspace(grass.cgrad_workspace(T, m, n, r, grass.BF16)))
    want = dict(GC=GC, M=M.clone(), V=V.clone(), W=W.clone())
    grass.adam_scatter(GC, want["M"], want["V"], lr, b1, b2, eps, t, want["W"], idx, rho, -0.7)
    got = dict(GC=torch.empty_like(GC), M=M, V=V, W=W)
    grass.step_group([dY], X, [idx], [rho], [M], [V], [W], lr, b1, b2, eps, t, -0.7,
                     grass.workspace(grass.step_group_workspace(T, n, [r], grass.BF16)),
                     GCs=[got["GC"]] if keep else None)
    if not keep:
        del want["GC"]
    _same(got, want)


# rows and columns of W around the update's 64 x 64 tiles
@pytest.mark.parametrize("mrows", [1, 61, 64, 129, 1027])
@pytest.mark.parametrize("r,repeat", [(1, False), (63, True), (64, False), (130, True), (130, False)])
@pytest.mark.parametrize("slices,sdt", [(2, torch.float32), (12, torch.bfloat16)])
def test_columns(mrows, r, repeat, slices, sdt):
    T, m = 2592, 200
    grass.set_test_option(grass.TEST_MAX_K_SLICES, slices)
    dX, dYt, idx, rho, M, V, _ = _setup(T, m, mrows, r, torch.bfloat16, sdt, torch.bfloat16, 0, repeat)
    W = torch.randn(mrows, m, device=DEV).to(torch.bfloat16)
    lr, b1, b2, eps, t = ADAM
    GC = torch.empty(r, mrows, device=DEV)
    grass.compressed_grad(dX, dYt, idx, rho, GC,
                          grass.workspace(grass.cgrad_workspace(T, m, mrows, r, grass.BF16)))
    want = dict(M=M.clone(), V=V.clone(), W=W.clone(), U=torch.empty_like(GC))
    grass.adam_rows(GC, want["M"], want["V"], lr, b1, b2, eps, t, want["U"])
    ref_w = W.float()
    grass.scatter_update_cols(want["W"], idx, rho, 0.6, want["U"])
    # the column update itself: W is rounded once, half a bf16 ulp is at most 2^-8 of the value; the fp32
    # sum of a run (a few terms of size 0.02) is off by less than 1e-7
    add = torch.zeros(mrows, m, device=DEV, dtype=torch.float64)
    add.index_add_(1, idx.long(), (rho.double()[:, None] * want["U"].double()).T)
    exact = ref_w.double() + 0.6 * add
    assert ((want["W"].double() - exact).abs() <= 2.0 ** -8 * exact.abs() + 1e-6).all()
    got = dict(M=M, V=V, W=W, U=torch.empty_like(GC))
    grass.step_cols(dYt, dX, idx, rho, M, V, got["U"], W, lr, b1, b2, eps, t, 0.6,
                    grass.workspace(grass.step_cols_workspace(T, mrows, m, r, grass.BF16)))
    _same(got, want)
