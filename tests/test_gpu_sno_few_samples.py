"""The surrogate's kernels that take a block per sample, on either side of the batch size where
blocks and splits change, for inference and training.

A sample's result does not depend on the batch but for the order of FP64 sums over its pixels
(relative 1e-16 each) before they are rounded to FP32: densities within 1e-6 of their largest
value, as FP32 rounds them, and their sums within 1e-5 of one."""
import numpy as np
import pytest

from oracle import sno_reference as ref
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


@pytest.mark.parametrize("B", [3, 16, 24, 32])
def test_training_gradient_with_parts_of_either_form(B):
    """32^2 pixels: parts of 4 B rows, the width-32 kernel from 64 on in steps of 64, else the
    general product; against the FP64 gradient with the bounds of BF16 activations (cosine
    0.99, each 1x1 map within 10 % with sharp parameters)."""
    import torch
    cfg = ref.Config(S=32, C=32, M=16, L=2)
    d = ref.unpack(ref.random_params(cfg, 47, spectral_scale=4.0 / cfg.C), cfg)
    d["Wp"] = 8.0 * d["Wp"]
    p = ref.pack(d, cfg).astype(np.float32)
    rng = np.random.default_rng(48)
    f = rng.standard_normal((B, 32, 32)) * 2.0 + 1.0
    rho = rng.dirichlet(np.ones(1024), size=B).reshape(B, 32, 32).astype(np.float32)
    net = _net(32, 32, 16, B, "bf16", True)
    try:
        net.set_params(p)
        ft, rt = torch.from_numpy(f).cuda().contiguous(), torch.from_numpy(rho).cuda().contiguous()
        net.forward(ft)
        loss, g = net.backward(ft, rt, want_grad=True)
    finally:
        net.close()
    lref, gref = ref.backward(p.astype(np.float64), f, rho.astype(np.float64), cfg)
    g64 = g.astype(np.float64)
    assert abs(loss - lref) < 0.02 * lref
    assert float(g64 @ gref / (np.linalg.norm(g64) * np.linalg.norm(gref))) > 0.99
    o = 0
    for name, shape in ref.param_layout(cfg):
        n = int(np.prod(shape))
        if name[0] == "W":
            assert np.linalg.norm(g64[o:o + n] - gref[o:o + n]) < 0.1 * np.linalg.norm(gref[o:o + n]), name
        o += n
