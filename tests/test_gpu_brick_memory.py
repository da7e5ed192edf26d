"""P's bricked copy is the library's own choice while p_layout is open, so a
solve or a batch that fits without it runs without it: from a workspace that
lacks its place, and on a device too small for it (a cube one voxel wide in
two directions, whose copy in bricks of 8 is 64 times its size).  The results
keep their bits."""
import numpy as np
import pytest

import tomo_synth as ts
from _gpu_common import need_gpu, to_dev

pytestmark = pytest.mark.gpu

LONG = 1 << 22  # voxels of the thin cube: its copy takes 1 GiB a frame


@pytest.fixture()
def tomo():
    t = need_gpu()
    t.autotune_clear()
    old = t.get_tuning()
    yield t
    t.set_tuning(**old)


def _thin(tomo, frames):
    """One view of 4 x 4 pixels a frame, looking across the long axis."""
    views, pix = ts.make_views(90.0 + 0.001 * np.arange(frames), (4, 4), 2.0)
    g = ts.Geometry((LONG, 1, 1), np.full(3, -1.5), np.full(3, 1.5), views, pix,
                    view_frame=np.arange(frames, dtype=np.int32), nframes=frames)
    dg = tomo.DeviceGeometry(g)
    assert tomo.class_tuning(dg)[0]["p_layout"] == 3
    return dg


def _x_fastest(tomo, f):
    old = tomo.set_tuning(p_layout=0)
    try:
        return f()
    finally:
        tomo.set_tuning(**old)


def test_workspace_without_the_copy(tomo):
    import torch

    views, pix = ts.make_views(7.0 + 15.0 * np.arange(24), (150, 141), 3.4)
    dg = tomo.DeviceGeometry(ts.Geometry((128, 104, 80), np.full(3, -1.5), np.full(3, 1.5), views, pix))
    assert tomo.class_tuning(dg)[0]["p_layout"] == 2
    y = to_dev(np.random.default_rng(1).normal(size=dg.npix))
    kw = dict(lam_r=1e-2, max_iter=6)
    full = tomo.cg_workspace_bytes(dg, max_iter=6)
    least = _x_fastest(tomo, lambda: tomo.cg_workspace_bytes(dg, max_iter=6))
    assert full - least >= 4 * dg.nvox
    ref = _x_fastest(tomo, lambda: tomo.cg_solve(dg, y, **kw)[0]).clone()
    for size in (least, full - 256, full):
        ws = torch.empty(size, dtype=torch.uint8, device="cuda")
        assert torch.equal(tomo.cg_solve(dg, y, workspace=ws, **kw)[0], ref)
    with pytest.raises(RuntimeError, match="needed"):
        tomo.cg_solve(dg, y, workspace=torch.empty(least - 1, dtype=torch.uint8, device="cuda"), **kw)
    # a copy that the caller asked for is not done without
    old = tomo.set_tuning(p_layout=2)
    try:
        with pytest.raises(RuntimeError, match="needed"):
            tomo.cg_solve(dg, y, workspace=torch.empty(least, dtype=torch.uint8, device="cuda"), **kw)
    finally:
        tomo.set_tuning(**old)


def test_solve_whose_copy_passes_the_device(tomo):
    import torch

    frames = int(torch.cuda.mem_get_info()[1] >> 30) + 8
    dg = _thin(tomo, frames)
    y = to_dev(np.random.default_rng(2).normal(size=dg.npix))
    kw = dict(lam_r=1e-2, lam_t=1.0, max_iter=2)
    print(f"[thin] {frames} frames, copy of {frames} GiB", flush=True)
    x, rep = tomo.cg_solve(dg, y, **kw)
    assert rep["iters"] == 2
    ref, rep0 = _x_fastest(tomo, lambda: tomo.cg_solve(dg, y, **kw))
    assert float(ref.abs().max()) > 0
    assert torch.equal(x, ref)
    np.testing.assert_array_equal(rep["history"], rep0["history"])


def test_batch_whose_copies_pass_the_device(tomo):
    """Systems of one geometry share their input; together their copies are
    larger than the device."""
    import torch

    nsys = 16
    frames = int(torch.cuda.mem_get_info()[1] >> 30) // nsys + 1
    dg = _thin(tomo, frames)
    print(f"[thin batch] {nsys} systems of {frames} frames", flush=True)
    x = to_dev(np.random.default_rng(3).uniform(size=dg.cube_shape))
    ref = _x_fastest(tomo, lambda: tomo.project(dg, x)).clone()
    b = tomo.Batch([dg] * nsys)
    try:
        for img in b.project([x] * nsys):
            assert torch.equal(img, ref)
    finally:
        b.close()


def test_batch_gives_its_copies_back_to_a_solve(tomo):
    """The copies fit when the batch is created; later the device is too full
    for a solve's vectors beside them."""
    import torch

    nsys, frames = 4, 10
    dg = _thin(tomo, frames)
    y = to_dev(np.random.default_rng(4).normal(size=dg.npix))
    kw = dict(lam_r=1e-2, lam_t=1.0, max_iter=2, check_every=2)
    b = _x_fastest(tomo, lambda: tomo.Batch([dg] * nsys))
    ref = [v.clone() for v in b.cg_solve([y] * nsys, **kw)[0]]
    b.close()
    torch.cuda.synchronize()
    b = tomo.Batch([dg] * nsys)  # 40 GiB of copies
    torch.cuda.empty_cache()
    free = torch.cuda.mem_get_info()[0]
    fill = torch.empty(free - (3 << 29), dtype=torch.uint8, device="cuda")
    print(f"[thin batch] {fill.numel() >> 30} GiB taken, {torch.cuda.mem_get_info()[0] >> 20} MiB free", flush=True)
    try:
        xs, _ = b.cg_solve([y] * nsys, **kw)
        for v, r in zip(xs, ref):
            assert torch.equal(v, r)
        assert torch.cuda.mem_get_info()[0] > 30 << 30  # the copies' memory is free again
    finally:
        del fill
        torch.cuda.empty_cache()
        b.close()
