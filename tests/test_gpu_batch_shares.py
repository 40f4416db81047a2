"""Shares of a batch's cascade passes: laid out by the pass itself up to 256 problems and by
a kernel before it beyond.  Whatever the number of problems, each must match the FP64 oracle
run of that problem alone (relative L1 <= 1e-12, the same evaluations), eager and replayed."""
import numpy as np
import pytest

import gpmood_inputs as gi
import oracle

pytestmark = pytest.mark.gpu

SIZES = [(16, 12), (24, 24), (9, 20), (40, 33)]


@pytest.mark.parametrize("nprob,use_graph", [(1, False), (2, True), (64, False), (65, True), (256, True), (257, True), (300, False)])
def test_any_number_of_problems(nprob, use_graph):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2110_08683_amd import GPMoodBatch
    print(f"[gpu-case] batch shares nprob={nprob} graph={use_graph}", flush=True)
    kinds = len(SIZES)
    U0 = [gi.noise(nx, ny, seed=k) for k, (nx, ny) in enumerate(SIZES)]
    ref = [oracle.Oracle(nx, ny, bc=(1, 1), cascade=(3, 2, 1, 0)).run(U0[k], cfl=0.8, nsteps=2)
           for k, (nx, ny) in enumerate(SIZES)]
    b = GPMoodBatch([SIZES[p % kinds] for p in range(nprob)], bc=(1, 1), prec="f64", cascade=(3, 2, 1, 0), device="cuda:0")
    for p in range(nprob):
        b.gpm_batch_init_state(p, U0[p % kinds])
    for _ in range(2):
        b.gpm_batch_step(0.8, 1, use_graph=use_graph)
    iters, dts = b.gpm_batch_status()
    for p in range(nprob):
        Uo, dto, co, io = ref[p % kinds]
        U = b.gpm_batch_get_state(p)
        for v in range(4):
            assert np.abs(U[v] - Uo[v]).sum() <= 1e-12 * np.abs(Uo[v if v in (0, 3) else 0]).sum(), (p, v)
        assert iters[p] == io[-1, 2] and abs(dts[p] - dto[-1]) <= 1e-12 * dto[-1], p
    b.close()
