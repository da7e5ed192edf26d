"""P's three walks through the x-fastest cube (the machine loop, and the
compiler's loops for launches of few wavefronts and for sparse lines of sight)
sum the same segments in the same order as the walk from bricks: the same
bits, with masks, frames, gains and the obstacle."""
import numpy as np
import pytest

import tomo_synth as ts
from _gpu_common import need_gpu, to_dev

pytestmark = pytest.mark.gpu

FOUR, TWO, FEW = 0, 1, 2


def _geom(n, nviews, npix, lat=0.0, **kw):
    views, pix = ts.make_views(7.0 + 360.0 / nviews * np.arange(nviews), npix, 3.4, lat=lat)
    return ts.Geometry(n, np.array([-1.5, -1.4, -1.2]), np.array([1.3, 1.5, 1.4]), views, pix, **kw)


def _kernels(f):
    import torch
    from torch.profiler import ProfilerActivity, profile

    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        f()
        torch.cuda.synchronize()
    return [e.name for e in prof.events() if "k_project" in e.name]


CASES = [
    ((64, 64, 64), 8, (82, 80), {}, FEW),  # 52480 lines of sight, 2^18 voxels
    ((64, 64, 64), 8, (82, 79), {}, FOUR),  # 51824
    ((64, 64, 63), 8, (82, 80), {}, FOUR),  # fewer voxels
    ((90, 97, 95), 15, (90, 75), {}, FEW),
    ((105, 61, 146), 4, (131, 107), {"obstacle": np.array([0.1, 0.0, -0.1, 0.8])}, FEW),
    ((105, 61, 146), 4, (131, 107), {"lat": 20.0, "mask": True}, FEW),
    ((70, 81, 66), 12, (90, 61), {"frames": 3, "gains": True, "mask": True}, FEW),
    ((120, 110, 100), 3, (60, 50), {}, TWO),
    ((120, 110, 100), 3, (60, 50), {"obstacle": np.array([0.1, 0.0, -0.1, 0.8]), "mask": True}, TWO),
    ((40, 40, 40), 5, (60, 61), {"frames": 5, "gains": True}, FOUR),
]


@pytest.mark.parametrize("n,nviews,npix,kw,walk", CASES)
def test_walks_give_the_bricks_bits(n, nviews, npix, kw, walk):
    import torch

    tomo = need_gpu()
    tomo.autotune_clear()
    rng = np.random.default_rng(n[0] + nviews)
    kw = dict(kw)
    frames, masked = kw.pop("frames", 1), kw.pop("mask", False)
    if frames > 1:
        kw.update(view_frame=(np.arange(nviews) % frames).astype(np.int32), nframes=frames)
    if kw.pop("gains", False):
        kw["gains"] = rng.uniform(0.5, 2.0, size=nviews)
    g = _geom(n, nviews, npix, **kw)
    if masked:
        g.data_mask = (rng.uniform(size=g.nrays) > 0.3).astype(np.uint8)
        g.map_mask = (rng.uniform(size=(n[2], n[1], n[0])) > 0.2).astype(np.uint8)
    dg = tomo.DeviceGeometry(g)
    x = to_dev(rng.normal(size=dg.cube_shape))
    got = torch.empty(dg.npix, device="cuda")
    old = tomo.set_tuning(p_layout=0)
    try:
        names = _kernels(lambda: tomo.project(dg, x, out=got))
        assert len(names) == 1 and f"XWalk){walk}" in names[0], names
        tomo.set_tuning(p_layout=3)
        ref = tomo.project(dg, x)
    finally:
        tomo.set_tuning(**old)
    assert torch.equal(got, ref)
    assert float(ref.abs().max()) > 0
