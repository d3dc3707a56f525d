"""The surrogate's kernels that take a block per sample, on either side of the batch size where
blocks and splits change, for inference and training.

A sample's result does not depend on the batch but for the order of FP64 sums over its pixels
(relative 1e-16 each) before they are rounded to FP32: densities within 1e-6 of their largest
value, as FP32 rounds them, and their sums within 1e-5 of one."""
import numpy as np
import pytest

from paper_2303_01471_amd import qhd as q

pytestmark = pytest.mark.gpu


def _net(S, C, M, B, precision, train):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    from paper_2303_01471_amd.sno import Surrogate
    q.load_library()
    return Surrogate(grid=S, width=C, modes=M, layers=2, max_batch=B, precision=precision, train=train, seed=5)


@pytest.mark.parametrize("S,C,M,precision", [(32, 32, 16, "bf16"), (64, 32, 16, "bf16"), (32, 32, 8, "bf16"), (32, 8, 4, "fp32")])
def test_one_sample_alone_and_in_batches(S, C, M, precision):
    import torch
    rng = np.random.default_rng(91)
    f = torch.from_numpy(rng.standard_normal((256, S, S)) * 2.0 + 1.0).cuda().contiguous()
    net = _net(S, C, M, 256, precision, False)
    try:
        one = net.forward(f[:1].contiguous()).clone()
        for B in (2, 255, 256):
            out = net.forward(f[:B].contiguous())
            torch.cuda.synchronize()
            assert float((out[0] - one[0]).abs().max()) <= 1e-6 * float(one[0].max())
            assert float((out.double().sum(dim=(1, 2)) - 1.0).abs().max()) <= 1e-5
    finally:
        net.close()
