"""Weight gradients beside values that are not finite: a gradient element is a
sum over pairs of voxels inside the volume (and, in the 16 -> 16 layer, over
data gradients that are not zero), so an infinite value leaves the elements
alone that it has no pair in."""
import numpy as np
import pytest

from _gpu_common import need_gpu, to_dev, to_host
from test_gpu_convnet import flat, rand_params, unflat

pytestmark = pytest.mark.gpu

INF = float("inf")


def _backward(params, x, gout):
    tomo = need_gpu()
    return unflat(to_host(tomo.ConvNet(x.shape).backward(to_dev(flat(params)), to_dev(x), to_dev(gout))))


def _live_params(seed):
    """Weights and biases above 0: every activation is, for inputs above 0."""
    return [np.abs(p) + 0.05 for p in rand_params(seed)]


def test_output_gradient_at_a_corner():
    """An infinite output gradient at the last voxel: the last layer's taps
    that step outside there keep the sum over the other voxels."""
    shape = (6, 19, 21)
    params = _live_params(1)
    rng = np.random.default_rng(2)
    x, gout = rng.uniform(0.1, 1.0, size=shape), rng.uniform(0.1, 1.0, size=shape)
    gout[-1, -1, -1] = 0.0
    gw3 = _backward(params, x, gout)[4]
    gout[-1, -1, -1] = INF
    got = _backward(params, x, gout)
    inside = np.zeros((3, 3, 3), dtype=bool)
    inside[:2, :2, :2] = True
    assert np.all(got[4][0][:, inside] == INF)
    np.testing.assert_array_equal(got[4][0][:, ~inside], gw3[0][:, ~inside])
    assert got[5][0] == INF
    # every tap of the layer below pairs a data gradient near the corner
    assert np.all(got[2] == INF) and np.all(got[3] == INF)


@pytest.mark.parametrize("axis", [0, 1, 2])
def test_thin_volumes(axis):
    """Volumes one voxel wide in two directions: the taps across them have no
    pairs, and their gradients are 0 beside an infinite output gradient."""
    shape = [1, 1, 1]
    shape[axis] = 5
    params = _live_params(3)
    x, gout = np.full(shape, 0.5), np.full(shape, 0.25)
    gout[0, 0, 0] = INF
    gw1, _, gw2, _, gw3, _ = _backward(params, x, gout)
    across = np.ones((3, 3, 3), dtype=bool)
    along = [1, 1, 1]
    along[axis] = slice(None)
    across[tuple(along)] = False
    for gw in (gw1, gw2, gw3):
        assert np.all(gw[:, :, across] == 0.0)
        assert np.all(gw[:, :, 1, 1, 1] == INF)


def test_infinite_input():
    """An infinite input at a corner of a thin volume: the first layer's taps
    across it keep 0."""
    params = _live_params(4)
    x, gout = np.full((1, 1, 5), 0.5), np.full((1, 1, 5), 0.25)
    x[0, 0, 0] = INF
    gw1 = _backward(params, x, gout)[0]
    across = np.ones((3, 3, 3), dtype=bool)
    across[1, 1, :] = False
    assert np.all(gw1[:, :, across] == 0.0)
    assert not np.isfinite(gw1[:, :, 1, 1, 0]).any()  # voxel 1's gradient times the infinite input


def test_dead_channel_beside_infinite_activations():
    """Hidden activations that overflow to infinity: a channel of the next
    layer that is off everywhere has no data gradient, and its weights'
    gradients are 0."""
    params = _live_params(5)
    params[0][:] = 2.0 ** 100
    params[2][3] = 0.0
    params[3][3] = -1.0
    x = np.full((3, 18, 20), 2.0 ** 33)
    gw2 = _backward(params, x, np.full(x.shape, 0.25))[2]
    assert np.all(gw2[3] == 0.0)
    assert not np.isfinite(gw2[0]).any()


@pytest.mark.parametrize("shape", [(6, 19, 21), (2, 40, 33)])
def test_all_pairs_again(shape):
    """One NaN in the output gradient: the last layer's elements against FP64.
    The second layer's weights are 0, so its activations are its biases and
    every sum is exact."""
    params = _live_params(6)
    params[2][:] = 0.0
    params[3][:] = np.arange(1, 17) / 4.0
    rng = np.random.default_rng(7)
    gout = rng.integers(-8, 9, size=shape).astype(np.float64)
    gout[-1, -1, -1] = np.nan
    got = _backward(params, np.full(shape, 0.5), gout)[4][0]
    pad = np.pad(np.ones(shape), 1)
    for t in np.ndindex(3, 3, 3):
        inside = pad[t[0]:t[0] + shape[0], t[1]:t[1] + shape[1], t[2]:t[2] + shape[2]] > 0
        ref = gout[inside].sum()
        for c in range(16):
            np.testing.assert_array_equal(got[(c,) + t], np.float32(ref * params[3][c]))
