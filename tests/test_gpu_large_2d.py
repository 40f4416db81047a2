"""The largest 2D grid (32768 x 32768: more than 2^31 - 1 faces, and more than 2^29 cells
lowered by the first pass): a repeated state gives, bit for bit, the repeated result of its
period (130 GB of device memory; states compared on the device)."""
import numpy as np
import pytest

import gpmood_inputs as gi

pytestmark = pytest.mark.gpu


def test_largest_grid():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < 160 << 30:
        pytest.skip("needs 160 GiB of free device memory")
    from paper_2110_08683_amd import GPMood
    n, period = 32768, 64
    print(f"[gpu-case] 2d large {n}^2 f32", flush=True)
    U0 = gi.noise(period, period, seed=3, sigma=1.0)
    ref = {}
    p = GPMood(period, period, hi=(period / 64, period / 64), prec="f32", cascade=(3, 2, 1, 0), device="cuda:0")
    p.slot(0).copy_(torch.tensor(U0))
    p.gpm_set_dt(0.3 / 64 / 8)
    p.gpm_stage_dev(0, p.slot(0), p.slot(0), p.slot(1))
    ref = p.slot(1).clone()
    counts, it = p.gpm_troubled_counts()
    order = torch.tensor(p.gpm_get_order_mask()).cuda()
    p.close()
    g = GPMood(n, n, hi=(n / 64, n / 64), prec="f32", cascade=(3, 2, 1, 0), device="cuda:0")

    def tiles(x):
        return x.view(n // period, period, n // period, period)

    for v in range(4):
        tiles(g.slot(0)[v]).copy_(torch.tensor(U0[v]).float().cuda()[None, :, None, :])
    g.gpm_set_dt(0.3 / 64 / 8)
    torch.cuda.synchronize()
    g.gpm_stage_dev(0, g.slot(0), g.slot(0), g.slot(1))
    reps = (n // period) ** 2
    big, itb = g.gpm_troubled_counts()
    print(f"[gpu-case]   counts {list(big)} evaluations {itb} / {list(counts)} {it}", flush=True)
    assert n * n - big[0] >= 1 << 29
    for v in range(4):
        assert bool((tiles(g.slot(1)[v]) == ref[v][None, :, None, :]).all()), v
    assert bool((tiles(g.gpm_order_ptr()) == order[None, :, None, :]).all())
    assert itb == it and [int(c) for c in big] == [int(c) * reps for c in counts]
    g.close()
    del g
    torch.cuda.empty_cache()
