"""First-pass marches of several rows in every form of the kernel (walls, inflow slit, both
solvers, top radius 1 to 3, unequal spacing): small grids run one row a march, which the
oracle tests cover; longer marches must give the same stage bit for bit."""
import numpy as np
import pytest

import gpmood_inputs as gi

pytestmark = pytest.mark.gpu

FORMS = {
    "periodic": dict(bc=(0, 0)), "outflow": dict(bc=(1, 1)), "walls": dict(bc=(2, 2)),
    "walls x": dict(bc=(2, 0)), "walls y": dict(bc=(1, 2)),
    "slit": dict(bc=(1, 1), slit=(3, 0.3, 0.6, (1.4, 0.0, 3.0, 1.0))),
    "slit and walls": dict(bc=(2, 1), slit=(1, 0.3, 0.6, (1.4, 0.0, 3.0, 1.0))),
}


@pytest.mark.parametrize("top", [1, 2, 3])
@pytest.mark.parametrize("solver", ["hllc", "hll"])
@pytest.mark.parametrize("form", sorted(FORMS))
def test_longer_marches(form, solver, top):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2110_08683_amd import GPMood
    nx, ny = 70, 41
    print(f"[gpu-case] march forms {form} {solver} top={top} {nx}x{ny}", flush=True)
    for prec in ("f64", "f32"):
        for hi in ((1.0, 1.0 * ny / nx), (1.0, 1.0)):  # equal and unequal spacing
            ref = None
            for rows in (0, 4, 7, 12, 64):
                g = GPMood(nx, ny, hi=hi, prec=prec, cascade=tuple(range(top, -1, -1)), solver=solver, device="cuda:0",
                           **FORMS[form])
                g.gpm_set_tuning(rows_per_wave=rows)
                U = torch.tensor(gi.noise(nx, ny, seed=5)).to(g.dtype).cuda()
                V = torch.tensor(gi.quadrants(nx, ny, seed=6)).to(g.dtype).cuda()
                g.gpm_compute_dt_dev(U, 0.4)
                got = []
                for s in (0, 1, 2):
                    out = torch.empty_like(U)
                    g.gpm_stage_dev(s, V, U, out)
                    got += [out.cpu().numpy(), g.gpm_get_order_mask()]
                ref = ref or got
                assert all(np.array_equal(a, b, equal_nan=True) for a, b in zip(got, ref)), (prec, hi, rows)
                g.close()


# a grid whose automatic length is the longest, 12 rows, in both precisions; the last march
# of a column runs 4
@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_longest_automatic_march(prec):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2110_08683_amd import GPMood
    nx, ny = 4000, 700
    print(f"[gpu-case] longest automatic march {nx}x{ny} {prec}", flush=True)
    ref = None
    for rows in (0, 4, 12, 64):
        g = GPMood(nx, ny, prec=prec, cascade=(3, 2, 1, 0), device="cuda:0")
        g.gpm_set_tuning(rows_per_wave=rows)
        U = torch.tensor(gi.noise(nx, ny, seed=2)).to(g.dtype).cuda()
        g.gpm_compute_dt_dev(U, 0.8)
        out = torch.empty_like(U)
        g.gpm_stage_dev(0, U, U, out)
        got = out.cpu().numpy(), g.gpm_get_order_mask()
        ref = ref or got
        assert all(np.array_equal(a, b, equal_nan=True) for a, b in zip(got, ref)), rows
        g.close()
