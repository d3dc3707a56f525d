"""A relaxed-QP instance's readouts are the same bits whatever batch it is in."""
import numpy as np
import pytest

import qhd_inputs
from paper_2303_01471_amd import qhd as q

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    q.load_library()


@pytest.mark.parametrize("dim,r,batch", [(5, 8, 40), (4, 8, 300), (3, 15, 30), (7, 4, 9)])
def test_relaxed_qp_readouts(dim, r, batch):
    import torch
    from paper_2303_01471_amd.rqp import RelaxedQP
    probs = qhd_inputs.qp_instances(2, dim, 62)

    def run(n):
        h = RelaxedQP(dim, r, n, 1e-2, 5, q.QHD_SCHED_NESTEROV, (1e-3, 0.0))
        for i in range(n):
            h.set_objective(i, *probs[i % 2])
        h.evolve()
        res, marg, prob, st, psi = h.observe(want_marginals=True, want_prob=True, want_psi=True)
        torch.cuda.synchronize()
        out = [(x["norm"], x["e_f"], x["p_min"]) for x in res], marg.cpu().numpy(), prob.cpu().numpy()
        h.close()
        return out

    one, many = run(2), run(batch)
    for i in range(batch):
        assert many[0][i] == one[0][i % 2]
        assert np.array_equal(many[1][i], one[1][i % 2]) and np.array_equal(many[2][i], one[2][i % 2])
