"""The network's marching kernels over volumes with more columns than planes
and with fewer, and over columns of 8 and of 16 rows: a voxel's output does not
depend on how its volume is dealt to workgroups."""
import numpy as np
import pytest

from _gpu_common import need_gpu, to_dev
from test_gpu_convnet import flat, rand_params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,around", [
    ((4, 100, 90), (60, 100, 90)),  # 42 columns of 4 planes, of 60
    ((6, 40, 40), (12, 40, 40)),  # 9 columns of 6 planes, of 12
    ((33, 33, 33), (60, 70, 33)),  # columns of 8 rows, of 16
    ((90, 17, 33), (90, 48, 33)),  # the same
    ((5, 40, 300), (14, 40, 300)),  # the same
])
def test_cut_of_the_volume_does_not_matter(shape, around):
    """A volume and a larger one that begins with the same data: three layers of
    3x3x3 reach three voxels, so those further from where the smaller one ends
    have the same bits."""
    import torch

    tomo = need_gpu()
    params = to_dev(flat(rand_params(61)))
    rng = np.random.default_rng(62)
    big = rng.normal(size=around)
    small = np.ascontiguousarray(big[:shape[0], :shape[1], :shape[2]])
    a = tomo.ConvNet(shape).forward(params, to_dev(small))
    b = tomo.ConvNet(around).forward(params, to_dev(big))
    keep = tuple(slice(0, m if m == n else m - 3) for m, n in zip(shape, around))
    assert torch.equal(a[keep], b[keep])
    assert float(a[keep].abs().max()) > 0
