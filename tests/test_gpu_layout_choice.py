"""The layout and bundle P takes while the tuning leaves them open: the same
bits as the x-fastest walk on both sides of the rule's lines, also under
stream capture, where the caller's array is walked."""
import numpy as np
import pytest

import tomo_synth as ts
from _gpu_common import need_gpu, to_dev

pytestmark = pytest.mark.gpu


def _geom(n, nviews, npix, **kw):
    views, pix = ts.make_views(7.0 + 360.0 / nviews * np.arange(nviews), npix, 3.4)
    return ts.Geometry(n, np.full(3, -1.5), np.full(3, 1.5), views, pix, **kw)


CASES = [
    ((128, 104, 80), 24, (150, 141), {}, 2),  # single calls take bricks from 6e7 steps on
    ((128, 104, 80), 4, (140, 131), {}, 2),  # at least 2^20 voxels, rows of 128 bytes
    ((107, 103, 97), 4, (150, 140), {}, 2),  # odd sides, pixels up to 2.5 per voxel
    ((128, 128, 64), 40, (70, 33), {}, 3),  # rays sparser than 0.7 voxels
    ((107, 103, 97), 1, (70, 33), {}, 0),  # fewer than 6 crossings per voxel
    ((107, 103, 97), 3, (400, 380), {}, 0),  # dense rays, rows off the line size
    ((100, 100, 100), 4, (140, 131), {}, 0),  # fewer than 2^20 voxels
    ((128, 104, 80), 4, (140, 131), {"obstacle": np.array([0.1, 0.0, 0.0, 0.8])}, 2),
]


@pytest.mark.parametrize("n,nviews,npix,kw,layout", CASES)
def test_open_layout_gives_the_x_fastest_bits(n, nviews, npix, kw, layout):
    import torch

    tomo = need_gpu()
    dg = tomo.DeviceGeometry(_geom(n, nviews, npix, **kw))
    assert tomo.class_tuning(dg)[0]["p_layout"] == layout
    x = to_dev(np.random.default_rng(5).normal(size=dg.cube_shape))
    got = tomo.project(dg, x)
    old = tomo.set_tuning(p_layout=0, p_bundle=4)
    try:
        ref = tomo.project(dg, x)
    finally:
        tomo.set_tuning(**old)
    assert torch.equal(got, ref)
    out = torch.zeros_like(ref)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        tomo.project(dg, x, out=out)
    for _ in range(3):
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, ref)
