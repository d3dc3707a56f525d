"""Relaxed QP: captured calls replayed where the host's bookkeeping and the device part ways:
after a reset between capture and replay, and after an eager call of either parity.

The recorded steps are those of an eager call, so a replay from phi_0 is compared bitwise; a
recorded call that starts on the other set of axes than the eager one rounds in another order,
within 1e-6 (as in the other tests of replays)."""
import numpy as np
import pytest

import qhd_inputs
from paper_2303_01471_amd import qhd as q

pytestmark = pytest.mark.gpu

# one set of axes, two, three
LATTICES = [(3, 8), (5, 8), (8, 5)]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    q.load_library()


def _handle(dim, r, batch, nsteps, sched, p):
    from paper_2303_01471_amd.rqp import RelaxedQP
    h = RelaxedQP(dim, r, batch, 1e-2, nsteps, sched, p)
    for i, (Q, b) in enumerate(qhd_inputs.qp_instances(batch, dim, 61)):
        h.set_objective(i, Q, b)
    return h


def _capture(h, n):
    import torch
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):
        h.evolve(n, side)
    return g


def _density(h):
    import torch
    res, marg, prob, st, _ = h.observe(want_marginals=True, want_prob=True, want_psi=True)
    torch.cuda.synchronize()
    assert st == q.QHD_OK
    return res, marg.cpu().numpy(), prob.cpu().numpy()


@pytest.mark.parametrize("n", [1, 4, 5])
@pytest.mark.parametrize("dim,r", LATTICES)
def test_reset_between_capture_and_replay(dim, r, n):
    h = _handle(dim, r, 2, 12, q.QHD_SCHED_NESTEROV, (1e-3, 0.0))
    h.evolve(n)
    want, wmarg, wprob = _density(h)
    h.reset()
    g = _capture(h, n)
    for _ in range(2):
        h.reset()
        g.replay()
        res, marg, prob = _density(h)
        assert np.array_equal(prob, wprob) and np.array_equal(marg, wmarg)
        for a, b in zip(res, want):
            assert a["e_f"] == b["e_f"] and a["p_min"] == b["p_min"] and a["norm"] == b["norm"]
    del g
    h.close()


@pytest.mark.parametrize("before,between", [(2, 1), (1, 1), (1, 2)])
@pytest.mark.parametrize("dim,r", LATTICES)
def test_eager_call_between_capture_and_replay(dim, r, before, between):
    h = _handle(dim, r, 2, 64, q.QHD_SCHED_CONST, (0.5, 3.0))
    h.evolve(before + between + 6)
    _, _, want = _density(h)
    h.reset()
    h.evolve(before)
    g = _capture(h, 3)
    h.evolve(between)
    g.replay()
    g.replay()
    _, _, prob = _density(h)
    assert np.max(np.abs(prob - want)) <= 1e-6
    del g
    h.close()
