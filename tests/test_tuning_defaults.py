"""The tuning calls can ask for the library's defaults: a call that sets one value leaves the
others automatic, and a tuned context or batch can go back."""
import numpy as np
import pytest

import gpmood_inputs as gi


def test_wrappers_default_to_automatic(monkeypatch):
    from paper_2110_08683_amd import binding as B
    calls = []

    class Library:
        def gpm_set_tuning(self, ctx, passes, rows, tail):
            calls.append((passes, rows, tail))
            return B.GPM_OK

        def gpm_batch_set_tuning(self, batch, rows):
            calls.append(rows)
            return B.GPM_OK

    monkeypatch.setattr(B, "lib", lambda: Library())
    g, b = B.GPMood.__new__(B.GPMood), B.GPMoodBatch.__new__(B.GPMoodBatch)
    g.ctx = b.b = None
    g.gpm_set_tuning(tail_threshold=16)
    g.gpm_set_tuning(rows_per_wave=8)
    g.gpm_set_tuning()
    b.gpm_batch_set_tuning()
    assert calls == [(0, 0, 16), (0, 8, 32), (0, 0, 32), 0]


def _first_pass_us(g, torch):
    """The shortest first pass of 40 stages."""
    U = torch.tensor(gi.density_wave(64, 64)).to(g.dtype).cuda()
    out, best = torch.empty_like(U), np.inf
    g.gpm_set_dt(1e-3)
    for _ in range(40):
        g.gpm_instrument(1)
        g.gpm_stage_dev(0, U, U, out)
        best = min(best, g.gpm_instrument_read()["first_pass_ms"] * 1e3)
    g.gpm_instrument(0)
    return best


# 64^2 FP64: marches of 12 rows take 4.7 times the automatic length's time
@pytest.mark.gpu
def test_a_context_goes_back_to_the_defaults():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2110_08683_amd import GPMood
    from paper_2110_08683_amd.binding import GpmError
    print("[gpu-case] tuning back to the defaults, 64^2 f64", flush=True)
    g = GPMood(64, 64, prec="f64", cascade=(3, 2, 1, 0), device="cuda:0")
    fresh = _first_pass_us(g, torch)
    g.gpm_set_tuning(8, 12, 32)
    long = _first_pass_us(g, torch)
    g.gpm_set_tuning(tail_threshold=32)
    back = _first_pass_us(g, torch)
    print(f"[gpu-case]   first pass, us: fresh {fresh:.1f}, 12 rows {long:.1f}, back {back:.1f}", flush=True)
    assert back < 2 * fresh < long
    for bad in ((-1, 0, 32), (129, 0, 32), (0, 3, 32), (0, -4, 32), (0, 257, 32), (0, 0, -1), (0, 0, 4097)):
        with pytest.raises(GpmError):
            g.gpm_set_tuning(*bad)
    g.close()


@pytest.mark.gpu
def test_a_batch_goes_back_to_the_defaults():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2110_08683_amd import GPMoodBatch
    from paper_2110_08683_amd.binding import GpmError
    sizes = [(64, 40), (33, 57), (96, 96)]
    print(f"[gpu-case] batch tuning back to the defaults, sizes={sizes}", flush=True)
    ref = None
    for tune in (lambda b: None, lambda b: b.gpm_batch_set_tuning(12), lambda b: b.gpm_batch_set_tuning(),
                 lambda b: b.gpm_batch_set_tuning_per_problem([0, 7, 0])):
        b = GPMoodBatch(sizes, bc=(1, 1), prec="f32", cascade=(3, 2, 1, 0), device="cuda:0")
        for k, (nx, ny) in enumerate(sizes):
            b.gpm_batch_init_state(k, gi.quadrants(nx, ny, seed=k))
        tune(b)
        b.gpm_batch_step(0.8, 2, use_graph=True)
        got = [b.gpm_batch_get_state(k) for k in range(len(sizes))]
        ref = ref or got
        assert all(np.array_equal(x, y) for x, y in zip(got, ref))
        for bad in (-1, 3, 257):
            with pytest.raises(GpmError):
                b.gpm_batch_set_tuning(bad)
            with pytest.raises(GpmError):
                b.gpm_batch_set_tuning_per_problem([12, bad, 12])
        b.close()
