"""The kinetic factor of the highest frequency of an axis, |n| = N / 2, by its own angle.

A state of that frequency along one axis and constant along the other, f = 0, CONST schedule:
after n steps the state is itself times exp(-i n dt a |k|^2 / 2), and an error of the factor is
repeated every step.  The factor is formed from its angle as every other one is: the angle
rounded to FP32 turns (|r| <= 1/2: half a unit in the last place is 2^-26 turns, 0.94e-7 rad) and
the transcendental unit's error (1.2e-7), so the phase is off by at most 2.2e-7 a step, beside
the FP32 rounding of the state (1e-7 a step at most and of no fixed sign: 1e-5 in 1000 steps)."""
import math

import numpy as np
import pytest

from paper_2303_01471_amd import qhd as q

pytestmark = pytest.mark.gpu

STEPS = 1000


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    q.load_library()


@pytest.mark.parametrize("axis", [0, 1], ids=["x", "y"])
@pytest.mark.parametrize("flags,shape", [(0, (8, 8)), (0, (16, 32)), (0, (64, 16)), (0, (128, 128)), (0, (256, 64)),
                                         (0, (512, 512)), (q.QHD_OPT_RESIDENT, (32, 32)), (q.QHD_OPT_RESIDENT, (128, 64))])
def test_phase_of_the_highest_frequency(shape, flags, axis):
    import torch
    ny, nx = shape
    n = nx if axis == 0 else ny
    alpha = 0.02 + 0.47 * np.random.default_rng(17).random(40)  # turns of the factor, one instance each
    dt = 1e-3
    # phase per step in turns: pi dt a (n / 2)^2 on the unit box
    amps = alpha / (math.pi * dt * (n / 2) ** 2)
    count = 6 if n == 512 else len(alpha)
    specs = [q.InstanceSpec(shape=shape, nsteps=STEPS, dt=dt, sched=q.QHD_SCHED_CONST, sched_p=(float(a), 0.0))
             for a in amps[:count]]
    sign = (1.0 - 2.0 * (np.arange(n) % 2))
    z = (sign[None, :] if axis == 0 else sign[:, None]) * np.ones(shape)
    z = (z / math.sqrt(nx * ny)).astype(np.complex64)
    plan = q.Plan(specs, flags=flags)
    try:
        for i in range(count):
            plan.set_potential(i, np.zeros(shape))
            plan.set_state(i, z)
        plan.evolve()
        _, psi, _, st = plan.observe(want_psi=True)
        torch.cuda.synchronize()
        assert st == q.QHD_OK
        for i in range(count):
            got = plan.psi_of(psi, i).cpu().numpy().astype(np.complex128)
            turns = math.pi * dt * specs[i].sched_p[0] * (n / 2) ** 2 * STEPS
            phase = np.vdot(z.astype(np.complex128), got) * np.exp(2j * math.pi * math.fmod(turns, 1.0))
            assert abs(np.angle(phase)) <= STEPS * 2.2e-7 + 1e-5, (i, float(np.angle(phase)))
    finally:
        plan.close()
