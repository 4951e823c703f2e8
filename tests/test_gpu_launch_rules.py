"""The rules by which a transport launch takes its shape and its kinds of map
add, and what the run statistics say about them, on the GPU."""
import sys

import numpy as np
import pytest

import oracle
from paper_1711_03244_amd import mcx, workloads as W

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.mark.parametrize("variant", [0, 2])
@pytest.mark.parametrize("cap", [1, 3])
def test_events_count_every_live_iteration(cap, variant):
    """`events` counts lane iterations with a live photon: the segments, and
    for a photon that meets the cap the iteration that ends it."""
    p = W.cube_homogeneous(n=20).replace(src_pos=(9.5, 9.5, 0.0), max_events=cap)
    N = 3000
    say(f"[gpu] event cap {cap} variant {variant} N={N}")
    with mcx.Simulation(p, kernel_variant=variant) as sim:
        sim.run(N, 4)
        st = sim.stats()
    o = oracle.run(p, N, 4, nthreads=8)["counts"]
    assert st["capped"] == o["capped"] > 0
    assert st["events"] == o["events"] + o["capped"]
    assert st["scatters"] == o["scatters"] and st["face_events"] == o["face_events"]
    assert st["events"] == st["scatters"] + st["face_events"] + st["timeout"] + st["capped"]
