"""The batch autotuner never leaves a batch slower than it found it: where its choice is not
faster than the default march length the default stays, also for a batch that takes the
choice from the cache."""
import json
import types

import pytest

import gpmood_inputs as gi


def _stub(sizes, rows, gain, installed):
    """A batch without a device, whose autotuner answers rows and gain."""
    from paper_2110_08683_amd import GPMoodBatch
    b = GPMoodBatch.__new__(GPMoodBatch)
    b.b, b.sizes, b.prec, b.top, b.device, b.nprob = None, sizes, "f32", 3, "gpu", len(sizes)
    b.torch = types.SimpleNamespace(cuda=types.SimpleNamespace(get_device_name=lambda d: "MI355X"))
    b.gpm_batch_autotune = lambda cfl, reps: (list(rows), gain)
    b.gpm_batch_set_tuning_per_problem = lambda r: installed.append(list(r))
    return b


def test_cache_keeps_the_default_where_it_was_faster(tmp_path):
    cache, installed = str(tmp_path / "tune.json"), []
    assert _stub([(64, 64), (96, 96)], [4, 6], 1.0, installed).autotune(cache=cache) == ([4, 6], 1.0)
    assert _stub([(96, 96), (64, 64)], [], None, installed).autotune(cache=cache) == ([6, 4], None)
    assert installed == [[0, 0]]
    # a later sweep of a larger class that gained is applied, beside the marked ones
    _stub([(512, 512)], [16], 1.1, installed).autotune(cache=cache)
    assert _stub([(64, 64), (512, 512)], [], None, installed).autotune(cache=cache) == ([4, 16], None)
    assert installed[-1] == [0, 16]
    # and so does one that gained where an earlier one had not
    with open(cache) as f:
        table = json.load(f)
    del table[[k for k in table if k.endswith("c12")][0]]
    with open(cache, "w") as f:
        json.dump(table, f)
    _stub([(64, 64)], [8], 1.2, installed).autotune(cache=cache)
    _stub([(64, 64)], [], None, installed).autotune(cache=cache)
    assert installed[-1] == [8]


def test_an_older_cache_is_applied_as_before(tmp_path):
    cache, installed = str(tmp_path / "tune.json"), []
    with open(cache, "w") as f:
        json.dump({"MI355X|f32|r3|c12": 12}, f)
    assert _stub([(64, 64)], [], None, installed).autotune(cache=cache) == ([12], None)
    assert installed == [[12]]


# FP64 64^2: the default is one row a march, every candidate at least 1.5 times slower
@pytest.mark.gpu
@pytest.mark.parametrize("nprob", [1, 3])
def test_a_small_batch_keeps_its_march_length(nprob):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2110_08683_amd import GPMoodBatch
    print(f"[gpu-case] autotune of a small batch, {nprob} x 64^2 f64", flush=True)
    b = GPMoodBatch([(64, 64)] * nprob, bc=(1, 1), prec="f64", cascade=(3, 2, 1, 0), device="cuda:0")
    for k in range(nprob):
        b.gpm_batch_init_state(k, gi.quadrants(64, 64, seed=k))
    rows, gain = b.gpm_batch_autotune(0.8, reps=8)
    print(f"[gpu-case]   sweep's rows {rows}, gain {gain:.3f}", flush=True)
    assert gain >= 1.0
    b.close()
