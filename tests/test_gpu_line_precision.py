"""Where the lines of the alternating passes work in FP64.

The largest norm drift over the members of the 768-instance benchmark batch, per 10^4 steps, is
held to what separate passes along the two axes measured on the same batch (FP64 at the
frequency-space end of every column and at all four ends of 128-point rows): 5.45e-6 at 128^2,
5.20e-6 at 256^2.  Resident steps give the values of the streaming passes bit for bit."""
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest

import qhd_inputs
from gpu_helpers import note, run_gpu
from paper_2303_01471_amd import qhd as q

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    q.load_library()


@pytest.mark.parametrize("n,bar", [(128, 5.45e-6), (256, 5.20e-6)])
def test_norm_drift_of_the_batch(n, bar):
    members = [s for s in qhd_inputs.batched_2d(count=768) if s.shape[0] == n]
    specs = [q.InstanceSpec(shape=s.shape, nsteps=s.nsteps, dt=s.dt) for s in members]
    plan = q.Plan(specs)
    try:
        with ThreadPoolExecutor(8) as ex:
            for i, f in enumerate(ex.map(lambda s: s.grid(), members)):
                plan.set_potential(i, f)
        plan.evolve()
        res, _, _, st = plan.observe()
        assert st == q.QHD_OK
        rate = [abs(r["norm"] - 1.0) * 1e4 / s.nsteps for r, s in zip(res, specs)]
        note(f"  {len(specs)} x {n}^2: largest drift {max(rate):.2e} per 1e4 steps, median {np.median(rate):.2e}")
        assert max(rate) <= bar
    finally:
        plan.close()


@pytest.mark.parametrize("shape", [(128, 128), (32, 128), (128, 32), (64, 128), (128, 64)], ids=str)
@pytest.mark.parametrize("scheme", [q.QHD_SCHEME_STRANG, q.QHD_SCHEME_YOSHIDA4], ids=["strang", "yoshida4"])
def test_resident_steps_of_128_point_lines_are_bitwise_the_streaming_passes(shape, scheme):
    specs = [q.InstanceSpec(shape=shape, nsteps=k, dt=1e-2, scheme=scheme) for k in (41, 6)]
    fs = [qhd_inputs.landscape_grid(1600 + k, shape) for k in range(2)]
    a = run_gpu(specs, fs)[1]
    b = run_gpu(specs, fs, flags=q.QHD_OPT_RESIDENT)[1]
    for x, y in zip(a, b):
        assert np.array_equal(x, y)
