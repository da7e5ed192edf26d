"""P from bricks where the geometry's own rule takes them in single calls (6e7
voxel crossings and more): bricks of 4 and of 8, odd sides and an obstacle
against the x-fastest walk, bit for bit; and the x-fastest walk just below that
line and under stream capture."""
import numpy as np
import pytest

import tomo_synth as ts
from _gpu_common import need_gpu, to_dev
from test_gpu_x_walks import _kernels

pytestmark = pytest.mark.gpu

OBSTACLE = np.array([0.1, 0.0, 0.0, 0.8])


def _geom(n, nviews, npix, **kw):
    views, pix = ts.make_views(7.0 + 360.0 / nviews * np.arange(nviews), npix, 3.4)
    return ts.Geometry(n, np.full(3, -1.5), np.full(3, 1.5), views, pix, **kw)


@pytest.mark.parametrize("n,nviews,npix,kw,layout,steps", [
    ((128, 128, 64), 170, (70, 33), {}, 3, 6.2e7),  # rays sparser than 0.7 voxels
    ((107, 103, 97), 20, (150, 140), {}, 2, 6.4e7),  # odd sides
    ((107, 103, 97), 18, (150, 140), {}, 2, 5.8e7),  # too few crossings for a single call
    ((128, 104, 80), 24, (150, 141), {"obstacle": OBSTACLE}, 2, 7.9e7),
    ((131, 99, 85), 180, (60, 37), {"obstacle": OBSTACLE}, 3, 6.3e7),
])
def test_single_calls_on_both_sides_of_the_line(n, nviews, npix, kw, layout, steps):
    import torch

    tomo = need_gpu()
    tomo.autotune_clear()
    assert abs(0.5 * nviews * npix[0] * npix[1] * sum(n) / steps - 1.0) < 0.02
    dg = tomo.DeviceGeometry(_geom(n, nviews, npix, **kw))
    assert tomo.class_tuning(dg)[0]["p_layout"] == layout
    x = to_dev(np.random.default_rng(5).normal(size=dg.cube_shape))
    got = torch.empty(dg.npix, device="cuda")
    names = _kernels(lambda: tomo.project(dg, x, out=got))
    assert ["bricked" in s for s in names] == [steps >= 6e7], names
    old = tomo.set_tuning(p_layout=0)
    try:
        ref = tomo.project(dg, x)
    finally:
        tomo.set_tuning(**old)
    assert torch.equal(got, ref)
    # a captured call walks the caller's array: one kernel, no allocation
    out = torch.zeros_like(ref)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        tomo.project(dg, x, out=out)
    assert ["bricked" in s for s in _kernels(g.replay)] == [False]
    for _ in range(3):
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, ref)
