"""A sample's density is the same bits whatever batch it is in."""
import numpy as np
import pytest

from paper_2303_01471_amd import qhd as q

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    q.load_library()


@pytest.mark.parametrize("train", [False, True], ids=["inference", "training"])
@pytest.mark.parametrize("S,C,M,precision", [(32, 32, 16, "bf16"), (64, 32, 16, "bf16"), (32, 32, 8, "bf16"),
                                             (64, 8, 4, "fp32"), (32, 8, 4, "fp32")])
@pytest.mark.parametrize("offset", [1.0, 1e4])
def test_surrogate_density(S, C, M, precision, train, offset):
    """With a large offset the landscape's mean and variance cancel in FP64, so that the order of
    their sums shows in the FP32 features."""
    import torch
    from paper_2303_01471_amd.sno import Surrogate
    rng = np.random.default_rng(92)
    f = torch.from_numpy(rng.standard_normal((300, S, S)) * 2.0 + offset).cuda().contiguous()
    net = Surrogate(grid=S, width=C, modes=M, layers=2, max_batch=300, precision=precision, train=train, seed=5)
    try:
        full = net.forward(f).clone()
        for B in (1, 7, 255, 256):
            assert torch.equal(net.forward(f[:B].contiguous()), full[:B])
    finally:
        net.close()
