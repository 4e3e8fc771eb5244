"""The tail events of a step whose sets need two launches (rows on 16-byte boundaries, and rows that
are not) cover both of them."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_2406_17660_amd import grass
from gpu_util import DEV, rel_fro, to_f64, to_np
from test_gpu_parity import make_idx, randn

pytestmark = pytest.mark.gpu


def test_mixed_group_is_right_and_timed_over_both_launches():
    T, n, ms, rs = 256, 4096, (2048, 64), (960, 8)
    X = randn((T, n), torch.bfloat16, 1)
    dYs = [randn((T, m), torch.bfloat16, 2 + i, scale=0.1) for i, m in enumerate(ms)]
    host = [make_idx(m, r, 5 + i, False) for i, (m, r) in enumerate(zip(ms, rs))]
    idxs, rhos = ([torch.from_numpy(h[k]).to(DEV) for h in host] for k in range(2))
    Ms, Vs = ([torch.zeros((r, n), device=DEV) for r in rs] for _ in range(2))
    # the second W has an odd leading dimension: its rows take the one-element-per-lane form
    Ws = [torch.zeros((ms[0], n), device=DEV), randn((ms[1], n), torch.float32, 9, ld=n + 1)]
    W1 = to_f64(Ws[1]).copy()

    def tail_ms(count):
        ws = grass.workspace(grass.step_group_workspace(T, n, rs[:count], grass.BF16))
        events = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        for e in events:
            e.record()
        grass.step_group(dYs[:count], X, idxs[:count], rhos[:count], Ms[:count], Vs[:count], Ws[:count],
                         1e-3, 0.9, 0.999, 1e-8, 1, 0.5, ws, tail_events=events)
        torch.cuda.synchronize()
        return events[0].elapsed_time(events[1])

    tail_ms(2)
    for dY, (idx, rho), M in zip(dYs, host, Ms):
        assert rel_fro(to_f64(M), 0.1 * ref.compressed_grad(to_np(dY), to_np(X), idx, rho)) <= 2e-5
    # from zero moments U = -lr m^ / (sqrt(v^) + eps)
    U = -1e-3 * (to_f64(Ms[1]) / 0.1) / (np.sqrt(to_f64(Vs[1]) / 0.001) + 1e-8)
    W1[host[1][0]] += 0.5 * host[1][1][:, None] * U
    assert rel_fro(to_f64(Ws[1]), W1) <= 1e-6  # fp32 sums of W and an update of 1e-3 of it
    # the large set's launch comes first: the time of both is no less than that of it alone
    both, large = (min(tail_ms(count) for _ in range(10)) for count in (2, 1))
    assert both >= 0.8 * large, (both, large)
