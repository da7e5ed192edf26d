"""P^T where pixels are finer than voxels: neighbouring lanes take pixels 1, 2,
4 or 8 apart by the ratio of voxel to pixel; each pixel is walked once."""
import numpy as np
import pytest

import tomo_synth as ts
from _gpu_common import PT_RTOL, assert_p_close, length_resolution, need_gpu, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("masked", [False, True])
@pytest.mark.parametrize("ratio", [2.25, 2.35, 3.25, 3.35, 5.9, 6.1, 9.0])
def test_transpose_at_pixel_ratios(ora, ratio, masked):
    tomo = need_gpu()
    n = (13, 37, 10)
    ncol = int(round(ratio * 3.4 / np.mean(3.0 / np.array(n))))
    views, pix = ts.make_views(7.0 + 120.0 * np.arange(3), (ncol, ncol - 5), 3.4)
    g = ts.Geometry(n, np.full(3, -1.5), np.full(3, 1.5), views, pix)
    rng = np.random.default_rng(31)
    if masked:
        g.data_mask = (rng.random(g.nrays) < 0.7).astype(np.uint8)
    y = rng.normal(size=g.nrays).astype(np.float32).astype(np.float64)
    got = to_host(tomo.backproject(tomo.DeviceGeometry(g), to_dev(y), strategy=tomo.BP_BLOCKED))
    assert_p_close(got.reshape(-1), ora.backproject(g, y).reshape(-1), ora.backproject(g, np.abs(y)).reshape(-1),
                   rtol=PT_RTOL, what="P^T", atol=length_resolution(g) * np.abs(y).max())
