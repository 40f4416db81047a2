"""3D first evaluation on grids that are thin below the face axis, which take the line kernel
on y and z too: at the edges of that rule (16 cells a step, 32 columns) against the FP64 3D
oracle, one SSP-RK3 step within 1e-12 relative L1 (FP32 within 1e-4), the same final levels
and evaluations; and a thin grid takes no longer than the same cells laid along x."""
import time

import numpy as np
import pytest

import oracle
from tests.test_gpu_faces_3d import _state

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,bc", [((15, 4, 6), (0, 0, 0)), ((16, 5, 4), (1, 0, 1)), ((17, 4, 5), (0, 1, 0)),
                                  ((4, 4, 13), (1, 1, 0)), ((16, 2, 20), (1, 1, 1)), ((16, 2, 20), (0, 1, 0)),
                                  ((11, 3, 9), (0, 0, 1)), ((32, 1, 7), (0, 1, 0)), ((8, 2, 2), (1, 1, 1)),
                                  ((1, 1, 70), (1, 1, 0)), ((1, 70, 1), (1, 0, 1))])
def test_edges_of_the_line_kernel(n, bc):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2110_08683_amd import GPMood3D
    print(f"[gpu-case] 3d thin n={n} bc={bc}", flush=True)
    U0 = _state(n, seed=sum(n))
    Uo, dts, iters, counts = oracle.Oracle3D(n, bc=bc, cascade=(2, 1, 0)).run(U0, cfl=0.3, nsteps=1)
    for prec, tol in (("f64", 1e-12), ("f32", 1e-4)):
        g = GPMood3D(n, bc=bc, prec=prec, cascade=(2, 1, 0), device="cuda:0")
        g.gpm3_init_state(U0)
        g.gpm3_step(0.3, 1)
        U = g.gpm3_get_state()
        c, it = g.gpm3_troubled_counts()
        for v in range(5):
            scale = np.abs(Uo[v if v in (0, 4) else 0]).sum()
            assert np.abs(U[v] - Uo[v]).sum() <= tol * scale, (prec, v)
        if prec == "f64":
            assert list(c) == list(counts) and it == iters[-1, 2]
        g.close()


# marches whose 64 columns lie in as many rows, or are fewer than the lanes, took 1.5 to 1.9
# times the time of the same cells along x
@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_thin_grids_are_as_fast_as_long_ones(prec):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2110_08683_amd import GPMood3D
    us = {}
    for n in ((1, 8, 4000), (4000, 8, 1)):
        ext = [np.sin(2 * np.pi * (np.arange(k) + 0.5) / k) for k in n]
        r = 1.0 + 0.02 * (ext[2][:, None, None] + ext[1][None, :, None] + ext[0][None, None, :])
        m = [0.1 * r] * 3
        U0 = np.stack([r, *m, 2.5 + 0.5 * (m[0] ** 2 * 3) / r])
        g = GPMood3D(n, bc=(1, 1, 1), prec=prec, cascade=(2, 1, 0), device="cuda:0")
        best = []
        for _ in range(12):
            g.gpm3_init_state(U0)
            torch.cuda.synchronize()
            t = time.perf_counter()
            g.gpm3_step(0.3, 4)
            best.append((time.perf_counter() - t) / 4 * 1e6)
        us[n] = min(best)
        g.close()
    print(f"[gpu-case] thin against long, {prec}, us a step: {us}", flush=True)
    assert us[(1, 8, 4000)] <= 1.35 * us[(4000, 8, 1)]
