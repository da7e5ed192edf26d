"""P's shape and layout where the tuning leaves them to the geometry (p_layout
-1, the initial value) and where a caller or the autotuner has settled them:
which kernel a call then runs."""
import numpy as np
import pytest

import tomo_synth as ts
from _gpu_common import need_gpu, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture()
def tomo():
    t = need_gpu()
    t.autotune_clear()
    old = t.get_tuning()
    yield t
    t.set_tuning(**old)
    t.autotune_clear()


def _ring(tomo, n, nviews, npix):
    views, pix = ts.make_views(7.0 + 360.0 / nviews * np.arange(nviews), npix, 3.4)
    return tomo.DeviceGeometry(ts.Geometry(n, np.full(3, -1.5), np.full(3, 1.5), views, pix))


def _bricked(f):
    """Whether the calls of P in f() gather from bricks, from the names of the
    kernels they run."""
    import torch
    from torch.profiler import ProfilerActivity, profile

    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        f()
        torch.cuda.synchronize()
    names = [e.name for e in prof.events() if "k_project" in e.name]
    assert names, "no projection kernel seen"
    return ["k_project_bricked" in s for s in names]


SMALL = ((128, 104, 80), 4, (140, 131))  # bricks by the geometry's rule, 1.1e7 crossings


def test_initial_values_round_trip(tomo):
    dg = _ring(tomo, *SMALL)
    assert tomo.get_tuning()["p_layout"] == -1
    assert tomo.class_tuning(dg)[0]["p_layout"] == 2
    old = tomo.set_tuning(p_layout=3)
    tomo.set_tuning(**old)
    assert tomo.class_tuning(dg)[0]["p_layout"] == 2
    tomo.set_tuning(p_bundle=4)  # a bundle of the caller's own: the caller's array
    now = tomo.class_tuning(dg)[0]
    assert (now["p_bundle"], now["p_xcd_remap"], now["p_layout"]) == (4, 1, 0)


def test_x_fastest_can_be_asked_for(tomo):
    """(2, 1, 0) set by a caller is that walk, in a solve as in a call."""
    dg = _ring(tomo, (128, 104, 80), 24, (150, 141))  # 8e7 crossings
    x = to_dev(np.random.default_rng(1).normal(size=dg.cube_shape))
    assert _bricked(lambda: tomo.project(dg, x)) == [True]
    open_bytes = tomo.cg_workspace_bytes(dg, max_iter=5)
    tomo.set_tuning(p_bundle=2, p_xcd_remap=1, p_layout=0)
    now = tomo.class_tuning(dg)[0]
    assert (now["p_bundle"], now["p_xcd_remap"], now["p_layout"]) == (2, 1, 0)
    assert _bricked(lambda: tomo.project(dg, x)) == [False]
    assert open_bytes - tomo.cg_workspace_bytes(dg, max_iter=5) >= 4 * dg.nvox


def test_settled_bricks_are_walked_by_small_calls_too(tomo):
    """The rule that keeps short single calls off bricks is for the open
    choice: the same three fields set by a caller are honoured."""
    dg = _ring(tomo, *SMALL)
    x = to_dev(np.random.default_rng(2).normal(size=dg.cube_shape))
    assert _bricked(lambda: tomo.project(dg, x)) == [False]
    own = tomo.class_tuning(dg)[0]
    tomo.set_tuning(p_bundle=own["p_bundle"], p_xcd_remap=own["p_xcd_remap"], p_layout=own["p_layout"])
    assert _bricked(lambda: tomo.project(dg, x)) == [True]


BRICKS = ((128, 128, 128), 28, (256, 256))
ARRAY = ((128, 90, 80), 17, (190, 190))  # the same size class; fewer than 2^20 voxels
SPARSE = ((128, 128, 70), 30, (72, 60))  # bricks by its rule, and too short for a single call
TINY = ((70, 30, 20), 20, (70, 64))  # the class of SPARSE; every shape takes a launch's time


@pytest.mark.parametrize("tuned,other", [(BRICKS, ARRAY), (ARRAY, BRICKS), (TINY, SPARSE)])
def test_tuner_leaves_p_open_where_it_keeps_nothing(tomo, tuned, other):
    """Where no candidate beats the geometry's own choice, the other geometries
    of its size class keep to their own rule; a pick that is kept is what every
    call of the class runs, short ones too."""
    a, b = _ring(tomo, *tuned), _ring(tomo, *other)
    keys = ("p_bundle", "p_xcd_remap", "p_layout")
    own_a, own_b = [{k: tomo.class_tuning(g)[0][k] for k in keys} for g in (a, b)]
    assert (own_a["p_layout"] >= 2) != (own_b["p_layout"] >= 2)
    x = [to_dev(np.random.default_rng(4).normal(size=g.cube_shape)) for g in (a, b)]
    alone = [_bricked(lambda: tomo.project(g, v)) for g, v in zip((a, b), x)]
    chosen = {k: v for k, v in tomo.autotune(a, reps=5).items() if k in keys}
    print("P before and after tuning:", own_a, chosen, flush=True)
    (now_a, tuned_a), (now_b, tuned_b) = tomo.class_tuning(a), tomo.class_tuning(b)
    assert tuned_a and tuned_b
    assert {k: now_a[k] for k in keys} == chosen
    now = [_bricked(lambda: tomo.project(g, v)) for g, v in zip((a, b), x)]
    if chosen == own_a:
        assert {k: now_b[k] for k in keys} == own_b
        assert now == alone
    else:
        assert {k: now_b[k] for k in keys} == chosen
        assert now == [[chosen["p_layout"] >= 2]] * 2
