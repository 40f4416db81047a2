"""Schedule of a stage on the GPU: what a stage computes does not depend on how its first
pass is cut into marches, nor on where its cascade passes run or what an earlier stage
left in the pass lists (FP64 against the oracle, FP32 bit for bit between schedules)."""
import numpy as np
import pytest

import gpmood_inputs as gi
import oracle
from tests.parity_util import assert_fields_close

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    return torch


def _note(msg):
    print(f"[gpu-case] {msg}", flush=True)


def _context(n, bc, prec, cascade=(3, 2, 1, 0)):
    from paper_2110_08683_amd import GPMood
    return GPMood(n[0], n[1], bc=bc, prec=prec, cascade=cascade, device="cuda:0")


def _stage(torch, g, s, Un, Us):
    out = torch.empty_like(Us)
    g.gpm_stage_dev(s, Un, Us, out)
    return out.cpu().numpy(), g.gpm_get_order_mask().astype(np.int32)


# grids around the 62-column strips and the march lengths, down to the smallest a
# periodic axis takes; long and flat ones, and one that gets the longest marches
@pytest.mark.parametrize("n", [(4, 4), (62, 5), (63, 61), (125, 7), (5, 300), (640, 33), (2500, 1000)])
@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_march_length_does_not_change_a_stage(torch_cuda, n, prec):
    _note(f"march length {n} {prec}")
    torch = torch_cuda
    ref = None
    for rows in (None, 4, 7, 64):
        g = _context(n, (0, 0), prec)
        if rows is not None:
            g.gpm_set_tuning(rows_per_wave=rows)
        U = torch.tensor(gi.noise(n[0], n[1], seed=2)).to(g.dtype).cuda()
        g.gpm_compute_dt_dev(U, 0.8)
        got = _stage(torch, g, 0, U, U)
        if ref is None:
            ref = got
        assert np.array_equal(got[0], ref[0], equal_nan=True) and np.array_equal(got[1], ref[1]), (n, prec, rows)
        g.close()


# the pass lists hold entries of the stage before (any face of the grid) beyond the
# entries of this one
@pytest.mark.parametrize("bc", [(0, 0), (1, 1), (2, 2), (1, 2)])
@pytest.mark.parametrize("n", [(64, 64), (45, 67)])
def test_cascade_paths_after_a_longer_stage(torch_cuda, bc, n):
    _note(f"cascade paths after a longer stage {n} bc={bc}")
    torch = torch_cuda
    for prec in ("f64", "f32"):
        g = _context(n, bc, prec)
        big = torch.tensor(gi.noise(n[0], n[1], seed=9)).to(g.dtype).cuda()
        U = torch.tensor(gi.quadrants(n[0], n[1], seed=4)).to(g.dtype).cuda()
        ref = None
        for tail in (0, 32, 4096):
            g.gpm_set_tuning(tail_threshold=tail)
            g.gpm_compute_dt_dev(big, 0.8)
            _stage(torch, g, 0, big, big)
            dt = g.gpm_compute_dt_dev(U, 0.8)
            U1, _ = _stage(torch, g, 0, U, U)
            t1 = torch.tensor(U1).cuda()
            _stage(torch, g, 0, big, big)
            got = _stage(torch, g, 1, U, t1)
            if ref is None:
                ref = (U1,) + got
            assert all(np.array_equal(a, b) for a, b in zip(ref, (U1,) + got)), (prec, tail)
        if prec == "f64":
            o = oracle.Oracle(n[0], n[1], bc=bc)
            Uo, order, _, _ = o.stage(1, U.cpu().numpy(), ref[0], dt)
            assert np.array_equal(ref[2], order)
            assert_fields_close(ref[1], Uo)
        g.close()
