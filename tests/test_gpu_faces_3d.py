"""3D first evaluation on the GPU at grids around its wavefronts' edges (64 positions along
the rows on x, 64 columns and marches of up to 6 faces on y and z), down to one cell on an
axis, against the FP64 3D oracle: one SSP-RK3 step within 1e-12 relative L1 (the bound of
the other 3D cases), the same final levels and number of evaluations; FP32 within 1e-4."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def _state(n, seed):
    nx, ny, nz = n
    rng = np.random.default_rng(seed)
    r = 1.0 + 0.02 * rng.random((nz, ny, nx))
    m = [0.02 * r * (rng.random((nz, ny, nx)) - 0.5) for _ in range(3)]
    p = 1.0 + 0.02 * rng.random((nz, ny, nx))
    return np.stack([r, *m, p / 0.4 + 0.5 * (m[0] ** 2 + m[1] ** 2 + m[2] ** 2) / r])


@pytest.mark.parametrize("n,bc", [((3, 3, 3), (0, 0, 0)), ((61, 3, 4), (0, 0, 0)), ((62, 4, 3), (1, 0, 0)),
                                  ((63, 3, 3), (0, 1, 0)), ((65, 5, 3), (1, 1, 1)), ((4, 40, 5), (0, 0, 1)),
                                  ((5, 3, 37), (0, 0, 0)), ((13, 11, 12), (1, 0, 1)), ((1, 2, 30), (1, 1, 1)),
                                  ((130, 1, 2), (1, 1, 1))])
def test_first_evaluation_edges(n, bc):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2110_08683_amd import GPMood3D
    print(f"[gpu-case] 3d faces n={n} bc={bc}", flush=True)
    U0 = _state(n, seed=sum(n))
    o = oracle.Oracle3D(n, bc=bc, cascade=(2, 1, 0))
    Uo, dts, iters, counts = o.run(U0, cfl=0.3, nsteps=1)
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
