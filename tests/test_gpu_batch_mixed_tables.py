"""A batch in which some systems have a ray table and some cannot (a cube with a
side above 2^20 voxels): each system's P^T equals its own call, bit for bit, with
footprints by rows and without."""
import numpy as np
import pytest

import tomo_synth as ts
from _gpu_common import need_gpu, to_dev
from test_gpu_batch import _masked_frames, _ragged

pytestmark = pytest.mark.gpu


def _long():
    """A cube of 2^20 + 3 voxels in a row, seen from across."""
    views, pix = ts.make_views([88.0, 91.0], (20, 12), 2.6)
    return ts.Geometry(((1 << 20) + 3, 1, 1), np.full(3, -1.2), np.full(3, 1.2), views, pix)


def _fine(nviews, **kw):
    """Pixels finer than voxels: footprints by rows."""
    views, pix = ts.make_views(5.0 + 360.0 / nviews * np.arange(nviews), (60, 50), 3.2)
    return ts.Geometry((17, 20, 14), np.full(3, -1.4), np.full(3, 1.4), views, pix, **kw)


@pytest.mark.parametrize("rows", [False, True])
def test_batch_of_systems_with_and_without_a_table(rows):
    import torch
    from torch.profiler import ProfilerActivity, profile

    tomo = need_gpu()
    tomo.autotune_clear()
    geoms = [_long(), ts.tiny().geom, _masked_frames(), _ragged()]
    if rows:
        rng = np.random.default_rng(8)
        mask = (rng.uniform(size=4 * 60 * 50) > 0.3).astype(np.uint8)
        geoms = [_long()] + [_fine(k) for k in (3, 4, 5)] + [
            _fine(4, data_mask=mask), _fine(4, obstacle=np.array([0.0, 0.1, 0.0, 0.9]))]
    dgs = [tomo.DeviceGeometry(g) for g in geoms]
    rng = np.random.default_rng(9)
    imgs = [to_dev(rng.normal(size=dg.npix)) for dg in dgs]
    b = tomo.Batch(dgs)
    try:
        with profile(activities=[ProfilerActivity.CUDA]) as prof:
            b.backproject(imgs)
            torch.cuda.synchronize()
        names = [e.name for e in prof.events() if "k_batch_backproject" in e.name]
        assert len(names) == 1 and f"{str(rows).lower()}, (tomo::Rays)2" in names[0], names
        for _ in range(2):
            got = b.backproject(imgs)
            torch.cuda.synchronize()
            for k, dg in enumerate(dgs):
                ref = tomo.backproject(dg, imgs[k], strategy=tomo.BP_BLOCKED)
                assert torch.equal(got[k], ref), k
                assert float(ref.abs().max()) > 0
        xs, _ = b.cg_solve(imgs, lam_r=1e-2, max_iter=4, check_every=4)
        for k, dg in enumerate(dgs):
            x, _ = tomo.cg_solve(dg, imgs[k], lam_r=1e-2, max_iter=4, check_every=4, bp_strategy=tomo.BP_BLOCKED)
            assert torch.equal(xs[k], x), k
    finally:
        b.close()
