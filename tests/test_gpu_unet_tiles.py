"""The network's convolutions and weight gradients stage tiles of 16 x 4 x 4,
16 x 2 x 2 and 32 x 4 x 4 sites: boxes smaller than a tile (whose ring wraps
onto itself), one site over a tile's edge (at full, half and quarter
resolution) and several tiles with remainders, against the float64 oracle.

Bounds from the arithmetic, as in test_gpu_unet: every stored activation is
rounded to bfloat16 (2^-9 relative), 9 of them in the forward pass: 2e-2 of the
output's norm; the gradients pass through twice as many and a few ReLU gates
flip: 5e-2 of each tensor's norm, cosine above 0.998."""
import numpy as np
import pytest

from oracle import unet as oun
from tests.parity import rel_l2
from tests.test_gpu_unet import oracle_input, problem, to_dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SHAPES = [(4, 4, 4), (8, 4, 20), (12, 20, 36), (36, 8, 12), (20, 12, 68)]


@pytest.fixture(scope="module")
def ek():
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_1710_09421_amd import ek as binding
    binding.lib()
    return binding


@pytest.mark.parametrize("shape", SHAPES)
def test_forward_and_gradients_match_oracle(ek, shape):
    p, b, solid, y = problem(sum(shape), shape)
    c_out = 0.8
    x, s = oracle_input(b, solid)
    out, cache = oun.forward(p, x)
    inference = ek.UNet(shape, training=False)
    inference.set_params(oun.flatten(p), c_out)
    guess = torch.zeros(shape, dtype=torch.float64, device="cuda")
    inference.forward(to_dev(b), to_dev(solid, torch.uint8), guess)
    err = rel_l2(guess.cpu().numpy(), out[0] * s * c_out)
    print(shape, "forward", err)
    assert err < 2e-2
    net = ek.UNet(shape, training=True)
    net.set_params(oun.flatten(p), c_out)
    net.accumulate(to_dev(b), to_dev(solid, torch.uint8), to_dev(y * s * c_out))
    got, ref = oun.unflatten(net.gradient()), oun.backward(p, cache, out, y[None])
    for k in p:
        e = rel_l2(got[k], ref[k])
        cos = float(np.dot(got[k].ravel(), ref[k].ravel()) /
                    (np.linalg.norm(got[k]) * np.linalg.norm(ref[k])))
        print(shape, k, e, cos)
        assert e < 5e-2 and cos > 0.998, (k, e, cos)
