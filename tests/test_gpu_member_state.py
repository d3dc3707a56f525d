"""A member given a new state while its neighbours are anywhere in their runs: every member's
values are those of a plan of its own, bit by bit, whatever axis the others are on."""
import numpy as np
import pytest

import qhd_inputs
from gpu_helpers import run_gpu
from paper_2303_01471_amd import qhd as q

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    q.load_library()


@pytest.mark.parametrize("flags", [0, q.QHD_OPT_RESIDENT, q.QHD_OPT_NO_GRAPH], ids=["streaming", "resident", "no graph"])
@pytest.mark.parametrize("n", [(7, 6, 5), (140, 200, 3)], ids=str)
@pytest.mark.parametrize("model", [q.QHD_MODEL_QHD, q.QHD_MODEL_QAA], ids=["qhd", "qaa"])
def test_new_state_of_one_member_after_an_odd_call(n, flags, model):
    import torch
    shapes = [(64, 64), (64, 64), (32, 128)]
    kw = dict(model=model, sched=q.QHD_SCHED_LINEAR, sched_p=(10.0, 0.0)) if model == q.QHD_MODEL_QAA else {}
    specs = [q.InstanceSpec(shape=s, nsteps=k, dt=1e-2, **kw) for s, k in zip(shapes, n)]
    fs = [qhd_inputs.landscape_grid(1500 + k, s) for k, s in enumerate(shapes)]
    rng = np.random.default_rng(15)
    z = rng.standard_normal(shapes[0]) + 1j * rng.standard_normal(shapes[0])
    z = (z / np.linalg.norm(z)).astype(np.complex64)
    _, want, _, _ = run_gpu(specs, fs, flags=flags)
    _, fresh, _, _ = run_gpu(specs[:1], fs[:1], flags=flags, states={0: z})
    _, later, _, _ = run_gpu(specs[:1], fs[:1], flags=flags, states={0: z}, steps_done={0: 2})
    plan = q.Plan(specs, flags=flags)
    try:
        for i, f in enumerate(fs):
            plan.set_potential(i, f)
        for done, ref in ((0, fresh), (2, later)):
            plan.reset()
            plan.evolve(3)
            plan.set_state(0, z)
            plan.set_steps_done(0, done)
            plan.evolve(1)
            plan.observe()
            plan.evolve()
            _, psi, _, st = plan.observe(want_psi=True)
            torch.cuda.synchronize()
            assert st == q.QHD_OK
            got = [plan.psi_of(psi, i).cpu().numpy() for i in range(3)]
            assert np.array_equal(got[0], ref[0])
            for i in (1, 2):
                assert np.array_equal(got[i], want[i])
    finally:
        plan.close()
