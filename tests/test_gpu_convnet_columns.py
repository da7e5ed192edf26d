"""The network's marching kernels at the edges of their 16 x 16 columns and of
their z runs, against the FP64 oracle."""
import numpy as np
import pytest

from _gpu_common import need_gpu, to_dev, to_host
from test_gpu_convnet import BF16_REL, _abs_params, flat, rand_params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(1, 1, 1), (1, 16, 16), (2, 15, 17), (3, 31, 13), (5, 16, 32), (7, 33, 15),
                                   (40, 3, 33), (4, 17, 16)])
def test_forward_at_column_edges(ora, shape):
    """Per voxel within 8 x 2^-8 of the |.|-network: a few BF16 roundings (2^-9
    relative each) of the input, the weights and the two hidden activations."""
    tomo = need_gpu()
    params = rand_params(21)
    x = np.random.default_rng(22).normal(size=shape)
    got = to_host(tomo.ConvNet(shape).forward(to_dev(flat(params)), to_dev(x)))
    ref = ora.convnet_forward(params, x)
    bound = 8 * BF16_REL * ora.convnet_forward(_abs_params(params), np.abs(x)) + 1e-6
    assert np.all(np.abs(got - ref) <= bound)
