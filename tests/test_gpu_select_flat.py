"""Sampling without replacement at the sizes where the kernel's arrangement changes (groups of 64 rows,
64 / 128 / 256 groups in registers, the tree beyond): the draws are the oracle's bit for bit."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_2406_17660_amd import grass
from gpu_util import DEV, gpu_select, to_np

pytestmark = pytest.mark.gpu


def _statistic(m, law, seed):
    rng = np.random.default_rng(seed)
    if law == "spread":  # a few rows hold most of the weight: neighbouring draws hit one group
        s = np.exp(4.0 * rng.standard_normal(m))
    elif law == "zeros":  # most rows weigh the minimum (1)
        s = np.where(rng.random(m) < 0.9, 0.0, rng.random(m))
    else:
        s = np.full(m, 0.5)
    return s.astype(np.float32)


@pytest.mark.parametrize("m", [1, 2, 63, 64, 65, 1000, 4095, 4096, 4097, 8192, 8193, 13824, 16383, 16384, 16385])
@pytest.mark.parametrize("method,law", [(grass.SEL_MULTI_NORM, "spread"), (grass.SEL_MULTI_NORM2, "zeros"),
                                        (grass.SEL_UNIFORM, "equal")])
def test_draws_match_the_oracle(m, method, law):
    ref_method = {grass.SEL_MULTI_NORM: ref.MULTI_NORM, grass.SEL_MULTI_NORM2: ref.MULTI_NORM2,
                  grass.SEL_UNIFORM: ref.UNIFORM}[method]
    s = _statistic(m, law, m)
    t = torch.from_numpy(s).to(DEV)
    for r, scale in ((1, grass.SCALE_PAPER), (min(m, 65), grass.SCALE_INV_SQRT_RQ), (min(m, 1500), grass.SCALE_ONE)):
        idx, rho, status = gpu_select(t, r, method, False, scale, seed=977 + m, refresh_id=3)
        want_idx, want_rho, _ = ref.select_rows(s, r, ref_method, False, scale, 977 + m, 3)
        assert status == grass.OK
        assert np.array_equal(to_np(idx), want_idx)
        assert np.array_equal(to_np(rho), np.asarray(want_rho, np.float32))


@pytest.mark.parametrize("m", [64, 130, 5000])
def test_every_row_is_drawn_when_r_is_m(m):
    idx, rho, _ = gpu_select(torch.from_numpy(_statistic(m, "spread", 1)).to(DEV), m, grass.SEL_MULTI_NORM, False)
    assert np.array_equal(to_np(idx), np.arange(m)) and (to_np(rho) == 1).all()


@pytest.mark.parametrize("m", [4097, 4224, 4225, 8191, 8319, 16257])
@pytest.mark.parametrize("law", ["spread", "zeros", "equal"])
def test_two_rows_per_lane_match_the_oracle(m, law):
    """Groups of 128 rows: their edges, draws too close to a boundary for the rounded target (weights of 1)
    and, with equal weights in 16257 rows, the total past 2^53."""
    s = _statistic(m, law, m + 1)
    r = min(m, 2500)
    idx, rho, status = gpu_select(torch.from_numpy(s).to(DEV), r, grass.SEL_MULTI_NORM, False, grass.SCALE_INV_SQRT_RQ, seed=m)
    want_idx, want_rho, _ = ref.select_rows(s, r, ref.MULTI_NORM, False, grass.SCALE_INV_SQRT_RQ, m, 0)
    assert status == grass.OK and np.array_equal(to_np(idx), want_idx)
    assert np.array_equal(to_np(rho), np.asarray(want_rho, np.float32))


def test_every_row_of_groups_of_128_is_drawn():
    for m in (4500, 8400):
        idx, _, _ = gpu_select(torch.from_numpy(_statistic(m, "zeros", 2)).to(DEV), m, grass.SEL_MULTI_NORM2, False)
        assert np.array_equal(to_np(idx), np.arange(m))


@pytest.mark.parametrize("m,r", [(8192, 1), (8192, 67), (8192, 8192), (9001, 2), (9001, 131), (12345, 3000), (16384, 259)])
def test_totals_past_53_bits_are_drawn_in_integers(m, r):
    """Uniform draws, and draws of equal norms but for the last row's, from 8192 rows on: every remainder of four
    draws a turn, and all rows of the smallest such size."""
    s = _statistic(m, "equal", m)
    s[-1] *= 0.25
    for method, oracle in ((grass.SEL_UNIFORM, ref.UNIFORM), (grass.SEL_MULTI_NORM, ref.MULTI_NORM)):
        idx, _, status = gpu_select(torch.from_numpy(s).to(DEV), r, method, False, grass.SCALE_PAPER, seed=m + r)
        want, _, _ = ref.select_rows(s, r, oracle, False, grass.SCALE_PAPER, m + r, 0)
        assert status == grass.OK and np.array_equal(to_np(idx), want)
