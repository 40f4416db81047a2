"""Stage adjoint on the GPU where whole wavefronts of faces have the top radius (read with
compile-time positions and scalar weights) and where some do not: grids whose rows are
shorter and longer than a wavefront, all cells at the top order or a few lowered, against
central differences of the FP64 oracle's forced-order stage (1e-4 relative in FP64, the bar
of the other adjoint cases; FP32 within 1e-3 of the FP64 result in relative L1)."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def _smooth(nx, ny, rng):
    x, y = (np.arange(nx) + 0.5) / nx, (np.arange(ny) + 0.5) / ny
    X, Y = np.meshgrid(x, y)
    f = [sum(rng.uniform(-1, 1) * np.sin(2 * np.pi * (a * X + b * Y) + rng.uniform(0, 6)) for a in (0, 1) for b in (1, 2))
         for _ in range(4)]
    r, u, v, p = 1 + 0.1 * f[0], 0.4 + 0.1 * f[1], -0.3 + 0.1 * f[2], 1 + 0.1 * f[3]
    return np.stack([r, r * u, r * v, p / 0.4 + 0.5 * r * (u * u + v * v)])


@pytest.mark.parametrize("nx,ny,bc,lowered", [(64, 8, (0, 0), 0), (16, 40, (1, 1), 0), (70, 9, (0, 1), 3), (9, 70, (1, 0), 3),
                                              (130, 6, (1, 1), 1)])
def test_top_radius_adjoint(nx, ny, bc, lowered):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2110_08683_amd import GPMood
    print(f"[gpu-case] adjoint top {nx}x{ny} bc={bc} lowered={lowered}", flush=True)
    cascade, s = (3, 2, 1, 0), 1
    rng = np.random.default_rng(nx + ny)
    U, Us, lam = _smooth(nx, ny, rng), _smooth(nx, ny, rng), rng.standard_normal((4, ny, nx))
    mask = np.full((ny, nx), 3, dtype=np.int32)
    for t in range(lowered):
        mask[rng.integers(ny), rng.integers(nx)] = t % 3
    o = oracle.Oracle(nx, ny, bc=bc, cascade=cascade)
    dt = 0.3 / max(nx, ny)
    got = {}
    for prec in ("f64", "f32"):
        g = GPMood(nx, ny, bc=bc, prec=prec, cascade=cascade, device="cuda:0")
        dev = lambda a: torch.tensor(a, device="cuda:0").to(g.dtype)
        lUs, lUn = torch.empty_like(dev(U)), torch.zeros_like(dev(U))
        order = torch.tensor(mask.astype(np.uint8), device="cuda:0")
        dl = g.gpm_stage_vjp(s, dev(U), dev(Us), order, dt, dev(lam), lUs, lUn)
        got[prec] = (lUs.double().cpu().numpy(), lUn.double().cpu().numpy(), dl)
        g.close()
    lUs, lUn, dl = got["f64"]

    def phi(dUs=0.0, orc=o):
        return float((lam * orc.stage_forced(s, U, Us + dUs, dt, mask)).sum())

    v = rng.standard_normal((4, ny, nx))
    fd = (phi(1e-6 * v) - phi(-1e-6 * v)) / 2e-6
    ad = float((lUs * v).sum())
    assert abs(fd - ad) <= 1e-4 * max(abs(fd), np.abs(lUs * v).sum() * 1e-2)
    assert np.abs(lUn - 0.75 * lam).sum() <= 1e-12 * np.abs(lam).sum()
    h = 1e-5 * o.ell
    op, om = (oracle.Oracle(nx, ny, bc=bc, cascade=cascade, ell=o.ell + d) for d in (h, -h))
    fd = (phi(orc=op) - phi(orc=om)) / (2 * h)
    assert abs(fd - dl) <= 1e-4 * abs(fd)
    assert np.abs(got["f32"][0] - lUs).sum() <= 1e-3 * np.abs(lUs).sum()
