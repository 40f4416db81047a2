"""Who makes the claims of the cells the first pass lowered: their own kernel, or the tail
where the stage before needed no multi-block pass (unless there are too many: it hands back
and the kernel makes them).  A stage must not depend on it: against the FP64 oracle, and in
FP32 bit for bit against a context that always queues multi-block passes."""
import numpy as np
import pytest

import gpmood_inputs as gi
import oracle
from tests.parity_util import assert_fields_close

pytestmark = pytest.mark.gpu


def _state(n, kind):
    if kind == "noise":
        return gi.noise(*n, seed=3)
    U = np.zeros((4, n[1], n[0]))
    U[0], U[1], U[3] = 1.0, 0.3, 2.545
    if kind == "few":
        for j, i in ((0, 0), (n[1] // 2, n[0] - 1), (n[1] - 1, n[0] // 2)):
            U[0, j, i], U[3, j, i] = 3.0, 25.0
    return U


# the stages before it leave the next one to start on the tail ("calm"), with few claims
# or with more than the tail takes
@pytest.mark.parametrize("bc", [(0, 0), (1, 1), (2, 2)])
@pytest.mark.parametrize("n", [(24, 20), (65, 40)])
@pytest.mark.parametrize("seq", [("calm", "few"), ("calm", "noise"), ("few", "few", "noise", "few")])
def test_claims_by_the_tail(n, bc, seq):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2110_08683_amd import GPMood
    print(f"[gpu-case] first claims n={n} bc={bc} {seq}", flush=True)
    o = oracle.Oracle(n[0], n[1], bc=bc, cascade=(3, 2, 1, 0))
    for prec in ("f64", "f32"):
        g, h = (GPMood(n[0], n[1], bc=bc, prec=prec, cascade=(3, 2, 1, 0), device="cuda:0") for _ in range(2))
        h.gpm_set_tuning(8, 12, 32)
        for kind in seq:
            U0 = _state(n, kind)
            dt = 0.2 * min(1.0 / n[0], 1.0 / n[1]) / 6
            got = []
            for c in (g, h):
                U = torch.tensor(U0).to(c.dtype).cuda()
                out = torch.empty_like(U)
                c.gpm_set_dt(dt)
                c.gpm_stage_dev(0, U, U, out)
                counts, it = c.gpm_troubled_counts()
                got.append((out.cpu().numpy(), c.gpm_get_order_mask(), list(counts), it))
            assert np.array_equal(got[0][0], got[1][0], equal_nan=True) and np.array_equal(got[0][1], got[1][1]), kind
            assert got[0][2:] == got[1][2:], kind
            if prec == "f64":
                Uo, order, counts, it = o.stage(0, U0, U0, dt)
                assert np.array_equal(got[0][1], order) and got[0][3] == it, kind
                assert_fields_close(got[0][0], Uo, what=f"{kind} {n}")
        g.close()
        h.close()
