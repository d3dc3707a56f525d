"""Resident 128 x 32 and 32 x 128 instances on either side of the member count where the block
size changes: the line work and its order are the same, so states are compared bitwise."""
import numpy as np
import pytest

import qhd_inputs
from gpu_helpers import PSI_TOL, compare, run_gpu, run_oracle
from paper_2303_01471_amd import qhd as q

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("model", [0, 1], ids=["qhd", "qaa"])
@pytest.mark.parametrize("shape", [(128, 32), (32, 128)], ids=lambda s: "%dx%d" % s)
def test_either_block_size_gives_the_same_states(shape, model):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    kw = dict(model=q.QHD_MODEL_QAA, sched=q.QHD_SCHED_LINEAR, sched_p=(10.0, 0.0)) if model else {}
    fs = [qhd_inputs.landscape_grid(1900 + k, shape) for k in range(3)]
    specs = [q.InstanceSpec(shape=shape, nsteps=9, dt=1e-2, **kw) for _ in range(257)]
    _, few, _, _ = run_gpu(specs[:3], fs, flags=q.QHD_OPT_RESIDENT)
    res, many, _, _ = run_gpu(specs, [fs[i % 3] for i in range(257)], flags=q.QHD_OPT_RESIDENT)
    for i in (0, 1, 2, 255, 256):
        assert np.array_equal(many[i], few[i % 3])
    ref, ro = run_oracle(specs[0], fs[0])
    err, *_ = compare(specs[0], fs[0], res[0], many[0], ref, ro, f"{shape}")
    assert err <= PSI_TOL
