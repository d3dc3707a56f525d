"""1-D steps, every sub-step of a call in one launch: each line length (lines share a
wavefront up to 128 points), member counts that leave the last wavefront part empty,
members that stop at different steps, and split calls.

Tolerances: the state bar 1e-4 against the FP64 oracle; split calls are the same
arithmetic, so they are compared bitwise."""
import numpy as np
import pytest

import qhd_inputs
from gpu_helpers import PSI_TOL, compare, run_gpu, run_oracle
from paper_2303_01471_amd import qhd as q

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [8, 16, 32, 64, 128, 256, 512, 1024])
def test_members_of_uneven_lengths(n):
    """Steps around the 64 of a captured chunk; 9 members: a part-filled last block."""
    steps = (1, 2, 63, 64, 65, 7, 130, 3, 128)
    specs = [q.InstanceSpec(shape=(n,), nsteps=k, dt=2e-2) for k in steps]
    fs = [qhd_inputs.landscape_grid(1700 + k, (n,)) for k in range(len(steps))]
    res, psis, _, st = run_gpu(specs, fs)
    assert st == q.QHD_OK
    for i, (spec, f) in enumerate(zip(specs, fs)):
        ref, ro = run_oracle(spec, f)
        err, nd, d_ef, d_p = compare(spec, f, res[i], psis[i], ref, ro, f"{n}[{i}]")
        assert err <= PSI_TOL and d_ef <= 1e-4 and d_p <= 1e-4
    plan = q.Plan(specs)
    try:
        for i, f in enumerate(fs):
            plan.set_potential(i, f)
        for c in (1, 64, 3):
            plan.evolve(c)
            plan.observe()
        plan.evolve()
        _, psi, _, _ = plan.observe(want_psi=True)
        for i in range(len(specs)):
            assert np.array_equal(plan.psi_of(psi, i).cpu().numpy(), psis[i])
    finally:
        plan.close()
