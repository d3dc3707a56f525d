"""The alternating 2-D passes (one axis per step) where their bookkeeping can go wrong:
calls of odd length, which leave either axis owed, readouts between them, members that
stop at either parity, a captured odd-length evolve replayed (the device's axes then move
without the host), and meshes whose lines share a block with other instances.

Tolerances: the state bar 1e-4 against the FP64 oracle; split calls, readouts between calls
and the two ways to launch give the very same arithmetic, so they are compared bitwise.  A
replayed odd capture pays the owed operator in a launch of its own, one more rounding per
replay: against the plain run of the same steps within 1e-6 (as rounding orders are
compared elsewhere)."""
import numpy as np
import pytest

import qhd_inputs
from gpu_helpers import PSI_TOL, compare, note, run_gpu, run_oracle
from paper_2303_01471_amd import qhd as q

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    q.load_library()


SHAPES = [(8, 8), (16, 64), (64, 16), (32, 32), (128, 128), (8, 256), (256, 8), (64, 512), (512, 16), (1024, 8), (16, 1024)]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "%dx%d" % s)
def test_odd_calls_readouts_and_both_parities(shape):
    """Three members stop after 1, 6 and 9 steps: both axes are owed at the end."""
    steps = (9, 6, 1)
    specs = [q.InstanceSpec(shape=shape, nsteps=n, dt=2e-2) for n in steps]
    fs = [qhd_inputs.landscape_grid(1300 + k, shape) for k in range(3)]
    res, psis, _, st = run_gpu(specs, fs)
    assert st == q.QHD_OK
    for i, (spec, f) in enumerate(zip(specs, fs)):
        ref, ro = run_oracle(spec, f)
        err, nd, d_ef, d_p = compare(spec, f, res[i], psis[i], ref, ro, f"{shape}[{i}]")
        assert err <= PSI_TOL and d_ef <= 1e-4 and d_p <= 1e-4
    plan = q.Plan(specs)
    try:
        for i, f in enumerate(fs):
            plan.set_potential(i, f)
        for c in (1, 3, 1, 2):
            plan.evolve(c)
            plan.observe(want_psi=True)
        plan.evolve()
        _, psi, _, _ = plan.observe(want_psi=True)
        for i in range(3):
            assert np.array_equal(plan.psi_of(psi, i).cpu().numpy(), psis[i])
    finally:
        plan.close()


@pytest.mark.parametrize("flags", [0, q.QHD_OPT_RESIDENT], ids=["streaming", "resident"])
def test_replayed_odd_capture_continues_on_either_axis(flags):
    """evolve(3) captured and replayed four times, then an eager evolve: 15 steps."""
    import torch
    shapes = [(64, 64), (128, 64), (256, 256)]
    specs = [q.InstanceSpec(shape=sh, nsteps=15, dt=1e-2) for sh in shapes]
    fs = [qhd_inputs.landscape_grid(1350 + k, sh) for k, sh in enumerate(shapes)]
    _, want, _, _ = run_gpu(specs, fs, flags=flags)
    plan = q.Plan(specs, flags=flags)
    try:
        for i, f in enumerate(fs):
            plan.set_potential(i, f)
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=side):
            plan.evolve(3, stream=side)
        for _ in range(4):
            g.replay()
            torch.cuda.synchronize()
            plan.observe()
        plan.evolve()
        _, psi, _, st = plan.observe(want_psi=True)
        assert st == q.QHD_OK
        for i, (spec, f) in enumerate(zip(specs, fs)):
            got = plan.psi_of(psi, i).cpu().numpy()
            d = float(np.max(np.abs(got - want[i])))
            note(f"  {shapes[i]}: replayed vs plain max|dpsi| = {d:.2e}")
            assert d <= 1e-6
        del g
    finally:
        plan.close()


def test_qaa_stops_at_both_parities():
    specs = [q.InstanceSpec(shape=sh, nsteps=n, dt=1e-2, model=q.QHD_MODEL_QAA, sched=q.QHD_SCHED_LINEAR,
                            sched_p=(n * 1e-2, 0.0)) for sh in ((64, 64), (128, 128), (16, 256)) for n in (8, 5)]
    fs = [qhd_inputs.landscape_grid(1380 + k, s.shape) for k, s in enumerate(specs)]
    res, psis, _, st = run_gpu(specs, fs, chunks=[3])
    assert st == q.QHD_OK
    for i, (spec, f) in enumerate(zip(specs, fs)):
        ref, ro = run_oracle(spec, f)
        err, *_ = compare(spec, f, res[i], psis[i], ref, ro, f"qaa[{i}]")
        assert err <= PSI_TOL
