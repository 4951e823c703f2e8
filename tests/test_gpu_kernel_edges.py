"""Edges of the kernels' dispatch and of their exact sums on the GPU: the
sizes and launches where a split, a remainder or a carry can go wrong."""
import math
import sys

import numpy as np
import pytest

from paper_1711_03244_amd import mcx, workloads as W

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.mark.parametrize("adds", [mcx.MAP_ADDS_64, mcx.MAP_ADDS_32])
@pytest.mark.parametrize("window", [1, 18])
def test_window_carries_beside_direct_adds(window, adds):
    """2e6 photons down a column of four cells of which the LDS window holds
    only the first one or two: a lane whose window addition carried out of
    32 bits next adds to the map directly, and the carry must be booked
    exactly once.  Every cell's exact sum is known (FP32 visit sums of
    identical photons, rounded to 2^-20 units): N round(2^20 v) units."""
    p = W.slab_column(nz=4, mua=0.005, mus=0.0)
    N = 2_000_000
    say(f"[gpu] slab_column N={N} window={window} map adds {adds}")
    maps = []
    for w in (window, -1):
        with mcx.Simulation(p) as sim:
            sim.set_launch(1024, 64, w)
            sim.set_map_adds(adds)
            sim.run(N, 3)
            maps.append(sim.fluence(mcx.MCX_RAW, f64=True))
    assert np.array_equal(maps[0], maps[1])
    mua = float(p.media[1, 0])
    expect = (-math.expm1(-mua)) / mua
    for k in range(4):
        assert maps[0][0, k, 1, 1] / N == pytest.approx(math.exp(-k * mua) * expect, rel=2e-6)
