"""The network's gradient kernels at the edges of their columns (16 x 16, 32 x 8
and 64 x 16) and of their z runs, against the FP64 oracle."""
import numpy as np
import pytest

from _gpu_common import need_gpu, to_dev, to_host
from test_gpu_convnet import _assert_grads_close, _grad_bounds, flat, rand_params, unflat

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(1, 1, 1), (1, 16, 64), (2, 15, 63), (3, 17, 65), (5, 8, 32), (4, 9, 31), (2, 7, 33),
                                   (40, 3, 17), (33, 1, 2)])
def test_backward_at_column_edges(ora, shape):
    """Element by element within the rounding of the products' BF16 factors."""
    tomo = need_gpu()
    params = unflat(flat(rand_params(51)).astype(np.float32))
    rng = np.random.default_rng(52)
    x = rng.normal(size=shape).astype(np.float32).astype(np.float64)
    gout = rng.normal(size=shape).astype(np.float32).astype(np.float64)
    got = unflat(to_host(tomo.ConvNet(shape).backward(to_dev(flat(params)), to_dev(x), to_dev(gout))))
    _, acts = ora.convnet_forward(params, x, keep=True)
    ref = ora.convnet_backward(params, acts, gout)
    _assert_grads_close(got, ref, _grad_bounds(ora, params, x, np.abs(gout)), f"backward {shape}")
