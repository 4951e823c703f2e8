"""Limits of the denoiser's kernels on the GPU: operands that are not finite or
not aligned, and the memory a network holds."""
import sys

import numpy as np
import pytest

import test_gpu_nn as T

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def weight_gradient_by_taps(x, gy):
    """gw[t][ci][n] of a 3x3x3 layer in float64: per tap only the products of
    voxels inside the volume, none of padding."""
    gw = np.zeros((27, x.shape[3], gy.shape[3]))
    for t in range(27):
        d = (t // 9 - 1, t // 3 % 3 - 1, t % 3 - 1)
        xs = tuple(slice(max(k, 0), n + min(k, 0)) for k, n in zip(d, x.shape))
        gs = tuple(slice(max(-k, 0), n + min(-k, 0)) for k, n in zip(d, x.shape))
        a, b = x[xs].reshape(-1, x.shape[3]), gy[gs].reshape(-1, gy.shape[3])
        with np.errstate(invalid="ignore"):
            gw[t] = (a[:, :, None] * b[:, None, :]).sum(0)
    return gw


@pytest.mark.parametrize("value", [np.inf, np.nan])
@pytest.mark.parametrize("shape,ci,co", [((5, 6, 7), 8, 8), ((9, 8, 5), 24, 16), ((3, 4, 4), 40, 8),
                                         ((8, 9, 12), 16, 40), ((17, 7, 21), 8, 24),
                                         ((5, 6, 7), 32, 8)])
def test_weight_gradient_of_activations_not_finite(shape, ci, co, value):
    """One activation at the volume's far corner, and one at each far face, is
    not finite: exactly the taps that pair it with a gradient inside the volume
    are not finite, also where the tiles end past the volume.  The others
    within 1e-5 of the sum of the products' sizes."""
    t = T.torch()
    say("[gpu] not finite", value, shape, ci, co)
    rng = np.random.default_rng(7)
    nz, ny, nx = shape
    where = [(nz - 1, ny - 1, nx - 1, 1), (nz - 1, ny // 2, nx // 2, 3),
             (nz // 2, ny - 1, nx // 2, 5), (nz // 2, ny // 2, nx - 1, 7)]
    x = T.O.bf16(np.abs(rng.normal(size=shape + (ci,))))
    for v in where:
        x[v] = value
    gy = T.O.bf16(rng.uniform(0.5, 1.5, size=shape + (co,)))
    want = weight_gradient_by_taps(x, gy)
    assert 0 < np.isfinite(want).mean() < 1
    gw = t.empty((27, ci, co), device="cuda")
    gb = t.empty((co,), device="cuda")
    w = t.zeros((27, ci, co), device="cuda")
    T.nn.mcx_nn_layer_backward(T.nn.MCX_NN_CONV3, shape, ci, co, T.dev_bf16(x), w, T.dev_bf16(gy),
                               None, gw, gb)
    got = T.host(gw)
    assert np.array_equal(np.isfinite(got), np.isfinite(want))
    assert np.array_equal(np.isnan(got), np.isnan(want))
    ok = np.isfinite(want)
    assert np.all(np.abs(got - want)[ok] <= 1e-5 * want[ok] + 1e-30)
    size = gy.reshape(-1, co).sum(0)
    assert np.all(np.abs(T.host(gb) - size) <= 1e-5 * size)
