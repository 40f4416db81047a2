"""A 3D grid whose FP64 variables take more than 4 GiB each, which the first evaluation reads
through 64-bit offsets: a repeated state gives, bit for bit, the repeated result of its period
(157 GB of device memory; states compared on the device)."""
import numpy as np
import pytest

from tests.test_gpu_long_marches_3d import _state

pytestmark = pytest.mark.gpu


def test_64_bit_offsets():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < 180 << 30:
        pytest.skip("needs 180 GiB of free device memory")
    from paper_2110_08683_amd import GPMood3D
    period, reps = (32, 16, 3), (16, 32, 683)
    n = tuple(p * r for p, r in zip(period, reps))
    assert 8 * n[0] * n[1] * n[2] >= 1 << 32
    print(f"[gpu-case] 3d large n={n} f64", flush=True)
    bc, ncell = (0, 0, 0), n[0] * n[1] * n[2]
    p = GPMood3D(period, hi=tuple(k / 64 for k in period), bc=bc, prec="f64", cascade=(2, 1, 0), device="cuda:0")
    U0 = _state(period, seed=7)
    p.gpm3_init_state(U0)
    p.gpm3_step(0.3, 1)
    ref = torch.tensor(p.gpm3_get_state()).cuda()
    counts, it = p.gpm3_troubled_counts()
    p.close()
    g = GPMood3D(n, hi=tuple(k / 64 for k in n), bc=bc, prec="f64", cascade=(2, 1, 0), device="cuda:0")
    slot = -(-5 * ncell * 8 // 256) * 256

    def tiles(k):  # slot k as [variable][z repeat][z][y repeat][y][x repeat][x]
        u = g.state_buf[k * slot:k * slot + 5 * ncell * 8].view(torch.float64)
        return u.view(5, reps[2], period[2], reps[1], period[1], reps[0], period[0])

    tiles(0).copy_(torch.tensor(U0).cuda()[:, None, :, None, :, None, :])
    torch.cuda.synchronize()
    g.gpm3_step(0.3, 1)
    for v in range(5):
        assert bool((tiles(1)[v] == ref[v][None, :, None, :, None, :]).all()), v
    big, itb = g.gpm3_troubled_counts()
    assert itb == it and list(big) == [c * reps[0] * reps[1] * reps[2] for c in counts] and counts[1] > 0
    g.close()
    del tiles, g
    torch.cuda.empty_cache()
