"""The calls of the first-claims tests take the paths they are for: after a stage without
multi-block passes the tail makes the claims itself, or hands back before it when the first
pass lowered more cells than it takes."""
import pytest

from tests.test_gpu_first_claims import _state

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("bc", [(0, 0), (1, 1), (2, 2)])
def test_which_kernel_makes_the_claims(prec, bc):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2110_08683_amd import GPMood
    n = (65, 40)
    print(f"[gpu-case] first claims' route n={n} bc={bc} {prec}", flush=True)
    g = GPMood(n[0], n[1], bc=bc, prec=prec, cascade=(3, 2, 1, 0), device="cuda:0")
    g.gpm_set_dt(0.2 / 65 / 6)
    stats = {}
    for kind in ("calm", "few", "noise"):
        U = torch.tensor(_state(n, kind)).to(g.dtype).cuda()
        g.gpm_stage_dev(0, U, U, torch.empty_like(U))
        stats[kind] = g.gpm_cascade_stats()  # multi-block passes, tail passes, hand-backs
    print(f"[gpu-case]   {stats}", flush=True)
    assert stats["calm"] == (0, 0, 0)
    assert stats["few"][0] == 0 and stats["few"][1] >= 1 and stats["few"][2] == 0
    assert stats["noise"][0] >= 1 and stats["noise"][2] >= 1
    g.close()
