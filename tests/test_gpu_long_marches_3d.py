"""3D marches of more than one face (the states carried from face to face through LDS, the
loads of the next cell, a segment's end): these take grids of 4e5 cells and more.  A state
that repeats along an axis gives, bit for bit, the repeated result of its period, whose
marches are of one face (and which the other 3D tests compare with the oracle); the spacing
is 1/64 on every grid, so both run the same arithmetic."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _state(n, seed):
    """Random cells of order one, a fifth of them lowered."""
    nx, ny, nz = n
    rng = np.random.default_rng(seed)
    r = 0.5 + rng.random((nz, ny, nx))
    m = [0.5 * r * (rng.random((nz, ny, nx)) - 0.5) for _ in range(3)]
    p = 0.5 + rng.random((nz, ny, nx))
    return np.stack([r, *m, p / 0.4 + 0.5 * (m[0] ** 2 + m[1] ** 2 + m[2] ** 2) / r])


def _run(n, bc, prec, U):
    from paper_2110_08683_amd import GPMood3D
    g = GPMood3D(n, hi=tuple(k / 64 for k in n), bc=bc, prec=prec, cascade=(2, 1, 0), device="cuda:0")
    g.gpm3_init_state(U)
    g.gpm3_step(0.3, 2)
    out = g.gpm3_get_state(), g.gpm3_get_order_mask()
    g.close()
    return out


# faces a march on y and z: 6 (the last segments of one face and of three), 2, 4 (of two and
# of none); the march's axis periodic, or open with the other one repeated
@pytest.mark.parametrize("n,period,bc", [((34, 180, 200), (34, 6, 5), (0, 0, 0)), ((34, 180, 200), (34, 180, 5), (1, 1, 0)),
                                         ((34, 180, 200), (34, 6, 200), (0, 0, 1)), ((67, 80, 80), (67, 5, 80), (1, 0, 1)),
                                         ((67, 80, 80), (67, 80, 4), (1, 1, 0)), ((33, 129, 203), (33, 129, 7), (0, 1, 0)),
                                         ((33, 129, 203), (33, 3, 203), (0, 0, 1))])
@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_repeated_state(n, period, bc, prec):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[gpu-case] 3d long marches n={n} period={period} bc={bc} {prec}", flush=True)
    U0 = _state(period, seed=sum(n))
    reps = tuple(a // b for a, b in zip(n, period))[::-1]
    U, order = _run(n, bc, prec, np.tile(U0, (1,) + reps))
    Up, op = _run(period, bc, prec, U0)
    assert (op < 2).any() and (op == 2).any()
    assert np.array_equal(U, np.tile(Up, (1,) + reps)) and np.array_equal(order, np.tile(op, reps))
