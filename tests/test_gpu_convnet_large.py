"""The network beyond its usual sizes: activations past what one buffer
resource spans (2^27 voxels), which take layers 2 and 3 and the data gradient by
tiles, and planes with more columns than the weight gradients have workgroups."""
import numpy as np
import pytest

from _gpu_common import need_gpu, to_dev, to_host
from test_gpu_convnet import _assert_grads_close, _grad_bounds, flat, rand_params, unflat

pytestmark = pytest.mark.gpu


def test_more_than_2_27_voxels():
    """Three layers of 3x3x3 reach three voxels, and six with their gradients:
    the first and the last planes of the large volume have the bits of small
    ones that end elsewhere, and an output gradient in the first planes gives
    the small volume's parameter gradients (the same FP32 sums, added in FP64)."""
    import torch

    tomo = need_gpu()
    nz, ny, nx = 516, 512, 512
    assert nz * ny * nx > 1 << 27
    params = to_dev(flat(rand_params(71)))
    gen = torch.Generator(device="cuda").manual_seed(72)
    x = torch.randn((nz, ny, nx), generator=gen, device="cuda")
    net = tomo.ConvNet((nz, ny, nx))
    small = tomo.ConvNet((16, ny, nx))
    out = net.forward(params, x)
    assert torch.equal(out[:13], small.forward(params, x[:16].contiguous())[:13])
    assert torch.equal(out[-13:], small.forward(params, x[-16:].contiguous())[3:])
    assert float(out[:13].abs().max()) > 0
    dout = torch.zeros_like(x)
    dout[:9] = torch.randn((9, ny, nx), generator=gen, device="cuda")
    grad = to_host(net.backward(params, x, dout))
    ref = to_host(small.backward(params, x[:16].contiguous(), dout[:16].contiguous()))
    np.testing.assert_allclose(grad, ref, rtol=1e-6, atol=1e-6 * np.abs(ref).max())


@pytest.mark.parametrize("shape", [(1, 520, 512), (1, 1030, 1030)])
def test_more_columns_than_workgroups(ora, shape):
    """1040 columns of 32 x 8 for 512 workgroups, and 4225 of 16 x 16 for 4096:
    workgroups take several each.  Within the rounding of the products' BF16
    factors."""
    tomo = need_gpu()
    params = unflat(flat(rand_params(73)).astype(np.float32))
    rng = np.random.default_rng(74)
    x = rng.normal(size=shape).astype(np.float32).astype(np.float64)
    gout = rng.normal(size=shape).astype(np.float32).astype(np.float64)
    got = unflat(to_host(tomo.ConvNet(shape).backward(to_dev(flat(params)), to_dev(x), to_dev(gout))))
    _, acts = ora.convnet_forward(params, x, keep=True)
    ref = ora.convnet_backward(params, acts, gout)
    _assert_grads_close(got, ref, _grad_bounds(ora, params, x, np.abs(gout)), f"backward {shape}")
