"""A solve reads its tuning once: its buffers are sized for that tuning and
every launch goes by it, whatever another thread sets meanwhile."""
import threading

import numpy as np
import pytest

import tomo_synth as ts
from _gpu_common import need_gpu, to_dev

pytestmark = pytest.mark.gpu


def test_solves_while_another_thread_changes_the_layout():
    """Sides just past a multiple of 16: a copy in bricks of 16 takes 2.9
    times the memory of one in bricks of 4, and the x-fastest walk takes none.
    P's layout does not change the bits of the iterates."""
    import torch

    tomo = need_gpu()
    tomo.autotune_clear()
    views, npix = ts.make_views([12.0, 75.0, 140.0, 230.0, 310.0], (40, 33), 3.2)
    dg = tomo.DeviceGeometry(ts.Geometry((34, 17, 18), np.full(3, -1.4), np.full(3, 1.4), views, npix))
    y = to_dev(np.random.default_rng(3).normal(size=dg.npix))
    kw = dict(lam_r=1e-2, max_iter=12, bp_strategy=tomo.BP_BLOCKED)
    old = tomo.get_tuning()
    stop = threading.Event()

    def change():
        k = 0
        while not stop.is_set():
            tomo.set_tuning(p_layout=(2, 4, 0, 3)[k % 4])
            k += 1

    t = threading.Thread(target=change)
    try:
        tomo.set_tuning(p_layout=0)
        ref, rep = tomo.cg_solve(dg, y, **kw)
        ref = ref.clone()
        assert rep["iters"] == 12
        t.start()
        for _ in range(40):
            x, _ = tomo.cg_solve(dg, y, **kw)
            assert torch.equal(x, ref)
    finally:
        stop.set()
        if t.is_alive():
            t.join()
        tomo.set_tuning(**old)
