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


def layer_forward_backward(kind, shape, ci, co, seed):
    """One layer forward (FP32 output) and backward on the GPU against the
    FP64 oracle on the same BF16 inputs, within 1e-5 of the sums of absolute
    terms: FP32 accumulation of random signs errs by about sqrt(K) 2^-24 of
    them, 2.5e-6 for the longest reduction (K = 1755), and by K 2^-24 at
    most."""
    import test_gpu_nn as T
    t = T.torch()
    x, w, b = T.layer_case(kind, shape, ci, co, seed)
    wq = T.O.bf16(w)
    oshape = T.out_shape(kind, shape)
    xd, wd, bd = T.dev_bf16(x), T.dev_f32(w), T.dev_f32(b)
    y = t.empty(oshape + (co,), dtype=t.float32, device="cuda")
    T.nn.mcx_nn_layer_forward(T.KIND[kind], shape, ci, co, xd, wd, bd, None, relu=False, y=y,
                              y_f32=True)
    scale = T.abs_terms(kind, x, wq) + np.abs(b)
    assert np.all(np.abs(T.host(y) - T.FWD[kind](x, wq, b)) <= 1e-5 * scale + 1e-30)
    gy = T.O.bf16(np.random.default_rng(seed + 1).normal(size=oshape + (co,)))
    gx = t.empty(tuple(shape) + (ci,), dtype=t.float32, device="cuda")
    gw = t.full(w.shape, float("nan"), dtype=t.float32, device="cuda")
    gb = t.full((co,), float("nan"), dtype=t.float32, device="cuda")
    T.nn.mcx_nn_layer_backward(T.KIND[kind], shape, ci, co, xd, wd, T.dev_bf16(gy), gx, gw, gb)
    ref = T.BWD[kind](x, wq, gy)
    lim = T.BWD[kind](np.abs(x), np.abs(wq), np.abs(gy))[:2] + (np.abs(gy).reshape(-1, co).sum(0),)
    for got, want, sc in zip((gx, gw, gb), ref, lim):
        assert np.all(np.abs(T.host(got) - want) <= 1e-5 * sc + 1e-30)


@pytest.mark.parametrize("kind,ci,co", [("conv3", 33, 65), ("conv3", 64, 31), ("conv3", 1, 63),
                                        ("down", 5, 63), ("down", 32, 33), ("up", 65, 7)])
def test_weight_packs_at_tile_edges(kind, ci, co):
    """Channel counts around the packs' 32- and 64-wide tiles, after a call of
    a larger layer left NaN weights in the scratch memory they reuse: the
    packs' padding must be zero, not what was there."""
    import test_gpu_nn as T
    t = T.torch()
    x = t.zeros((4, 4, 4, 96), dtype=t.bfloat16, device="cuda")
    nan = t.full((27, 96, 128), float("nan"), device="cuda")
    y = t.empty((4, 4, 4, 128), dtype=t.float32, device="cuda")
    T.nn.mcx_nn_layer_forward(T.nn.MCX_NN_CONV3, (4, 4, 4), 96, 128, x, nan, None, y=y, y_f32=True)
    say("[gpu] layer", kind, ci, co)
    layer_forward_backward(kind, (4, 6, 4), ci, co, 11)


def test_scratch_is_shared_between_threads():
    """Two threads on streams of their own call layers of different sizes
    again and again: each call's scratch memory is its own while it runs."""
    import threading

    import test_gpu_nn as T
    t = T.torch()
    jobs = []
    for k, (ci, co) in enumerate([(64, 64), (32, 96)]):
        x, w, b = T.layer_case("conv3", (6, 8, 8), ci, co, 20 + k)
        jobs.append((T.dev_bf16(x), T.dev_f32(w), T.dev_f32(b), ci, co))
    want = []
    for x, w, b, ci, co in jobs:
        y = t.empty((6, 8, 8, co), device="cuda")
        T.nn.mcx_nn_layer_forward(T.nn.MCX_NN_CONV3, (6, 8, 8), ci, co, x, w, b, y=y, y_f32=True)
        want.append(y.clone())
    t.cuda.synchronize()
    bad = []

    def work(k):
        x, w, b, ci, co = jobs[k]
        s = t.cuda.Stream()
        y = t.empty((6, 8, 8, co), device="cuda")
        for _ in range(30):
            T.nn.mcx_nn_layer_forward(T.nn.MCX_NN_CONV3, (6, 8, 8), ci, co, x, w, b, y=y,
                                      y_f32=True, stream=s)
            if not t.equal(y, want[k]):
                bad.append(k)

    threads = [threading.Thread(target=work, args=(k,)) for k in (0, 1)]
    for th in threads:
        th.start()
    for th in threads:
        th.join()
    assert not bad


@pytest.mark.parametrize("channels,shape,nsym", [
    ((8, 16), (6, 8, 8), 8),            # the generic kernel's gathers of several images
    ((16, 128), (16, 16, 16), 8),       # ranges spread over workgroups for one image only
    ((32, 64), (32, 32, 32), 4),        # resident weights for several images only
    ((5, 33, 64), (12, 20, 20), 8),     # odd channels, remainders of tiles
    ((16, 32), (10, 6, 14), 2),         # nx != ny
    ((32, 64), (104, 104, 104), 8),     # two groups of images
])
def test_images_in_one_launch_equal_one_by_one(channels, shape, nsym):
    """The symmetries' images share each layer's launch: the same bits as
    the network applied to one image after another, mapped back and added in
    order."""
    import test_gpu_nn as T
    t = T.torch()
    say("[gpu] symmetries", channels, shape, nsym)
    _, flat = T.make_net(channels, shape, 31)
    noisy, _ = T.fluence_pair(shape, 32)
    with T.nn.Denoiser(channels, shape) as d:
        d.set_params(flat)
        x = T.dev_f32(noisy)
        acc = None
        for op in range(nsym):
            u = t.empty_like(x)
            d.forward(x if op == 0 else T.nn.mcx_nn_mirror_xy(x, op), u_out=u)
            inv = (4 | (op & 1) << 1 | (op & 2) >> 1) if op & 4 else op
            if inv:
                u = T.nn.mcx_nn_mirror_xy(u, inv)
            acc = u if acc is None else acc + u
        u_sym = t.empty_like(x)
        d.forward(x, u_out=u_sym, symmetries=nsym)
        t.cuda.synchronize()
    assert t.equal(u_sym, acc / nsym)


@pytest.mark.parametrize("shape,ci,co,skip,relu,f32,shift", [
    ((2, 2, 2), 32, 8, True, True, False, 0),      # fewer voxels than a wave's
    ((3, 5, 7), 64, 40, True, False, False, 0),    # remainders of voxels and of channels
    ((4, 6, 10), 128, 24, False, True, True, 0),   # FP32 output
    ((2, 4, 4), 256, 64, True, True, False, 0),
    ((3, 3, 5), 96, 32, True, True, True, 0),      # channel chunks read again for each class
    ((16, 24, 24), 64, 128, True, True, False, 0),  # 64 voxels a wave, remainder
    ((3, 5, 7), 64, 40, True, True, False, 3),     # operands off 16-byte alignment
    ((3, 5, 7), 64, 12, True, True, False, 0),     # channels not a multiple of 8
])
def test_up_layer_edges(shape, ci, co, skip, relu, f32, shift):
    """Stride-2 up layers against the oracle on BF16 operands: FP32 sums of ci
    products (1e-5 of the sum of their sizes), then one BF16 rounding (2^-8)
    unless the output is FP32."""
    import test_gpu_nn as T
    t = T.torch()
    say("[gpu] up", shape, ci, co, skip, relu, f32, shift)
    x, w, b = T.layer_case("up", shape, ci, co, 41)
    big = tuple(2 * s for s in shape)
    sk = T.O.bf16(np.random.default_rng(42).standard_normal(big + (co,))) if skip else None
    wq = T.O.bf16(w)

    def placed(a, dtype):
        buf = t.zeros(a.size + shift, dtype=dtype, device="cuda")
        v = buf[shift:].view(a.shape)
        v.copy_(t.from_numpy(np.ascontiguousarray(a)))
        return v

    y = placed(np.zeros(big + (co,), np.float32), t.float32 if f32 else t.bfloat16)
    T.nn.mcx_nn_layer_forward(T.nn.MCX_NN_UP, shape, ci, co, placed(x, t.bfloat16), T.dev_f32(w),
                              T.dev_f32(b), y=y, y_f32=f32, relu=relu,
                              skip=None if sk is None else placed(sk, t.bfloat16))
    ref = T.FWD["up"](x, wq, b)
    size = T.FWD["up"](np.abs(x), np.abs(wq), np.abs(b))
    if skip:
        ref, size = ref + sk, size + np.abs(sk)
    if relu:
        ref = np.maximum(ref, 0)
    got = y.float().cpu().numpy()
    lim = 1e-5 * size + (0 if f32 else 2.0 ** -8 * np.abs(ref))
    assert np.all(np.abs(got - ref) <= lim + 1e-30)


@pytest.mark.parametrize("kind,shape,ci,co,shift", [
    ("conv3", (3, 5, 7), 8, 8, 0),          # one partial tile, a quarter of the channel blocks
    ("conv3", (9, 8, 5), 40, 24, 0),        # two tiles along z, remainders everywhere
    ("conv3", (8, 8, 8), 72, 96, 0),        # planes of taps, one group: gw finished at once
    ("conv3", (16, 24, 28), 32, 40, 0),     # planes of taps, several groups
    ("conv3", (24, 40, 44), 64, 32, 0),     # all taps, several tiles a workgroup
    ("conv3", (8, 6, 10), 32, 12, 0),       # output channels not in eights
    ("conv3", (6, 6, 6), 32, 32, 3),        # operands off 16-byte alignment
    ("down", (2, 2, 2), 8, 8, 0),
    ("down", (6, 10, 14), 24, 72, 0),
    ("down", (32, 32, 40), 32, 24, 0),
    ("up", (1, 1, 1), 8, 8, 0),
    ("up", (5, 3, 7), 72, 24, 0),
    ("up", (16, 20, 16), 24, 40, 0),
    ("up", (4, 4, 4), 32, 32, 3),
])
def test_weight_gradient_edges(kind, shape, ci, co, shift):
    """Weight gradients where tiles, channel blocks and groups of partial sums
    have remainders, with and without the bias gradient, against the oracle
    on BF16 operands: FP32 sums over the voxels, 1e-5 of the sum of the products'
    sizes."""
    import test_gpu_nn as T
    t = T.torch()
    say("[gpu] weight gradient", kind, shape, ci, co, shift)
    x, w, _ = T.layer_case(kind, shape, ci, co, 51)
    gy = T.O.bf16(np.random.default_rng(52).normal(size=T.out_shape(kind, shape) + (co,)))

    def placed(a):
        buf = t.zeros(a.size + shift, dtype=t.bfloat16, device="cuda")
        v = buf[shift:].view(a.shape)
        v.copy_(t.from_numpy(np.ascontiguousarray(a)))
        return v

    ref = T.BWD[kind](x, T.O.bf16(w), gy)
    lim = T.BWD[kind](np.abs(x), np.abs(T.O.bf16(w)), np.abs(gy))
    for with_bias in (False, True):
        gw = t.full(w.shape, float("nan"), dtype=t.float32, device="cuda")
        gb = t.full((co,), float("nan"), dtype=t.float32, device="cuda") if with_bias else None
        T.nn.mcx_nn_layer_backward(T.KIND[kind], shape, ci, co, placed(x), T.dev_f32(w), placed(gy),
                                   None, gw, gb)
        assert np.all(np.abs(T.host(gw) - ref[1]) <= 1e-5 * lim[1] + 1e-30)
        if with_bias:
            size = np.abs(gy).reshape(-1, co).sum(0)
            assert np.all(np.abs(T.host(gb) - ref[2]) <= 1e-5 * size + 1e-30)


def test_gradients_accumulate():
    """A second pass over the same volume added to the gradients doubles them
    exactly (their sums are taken in a fixed order): weight gradients that
    go through partial sums and those finished in one launch."""
    import test_gpu_nn as T
    t = T.torch()
    channels, shape = (32, 64, 128), (16, 32, 16)
    _, flat = T.make_net(channels, shape, 61)
    noisy, clean = T.fluence_pair(shape, 62)
    say("[gpu] gradients", channels, shape)
    with T.nn.Denoiser(channels, shape) as d:
        d.set_params(flat)
        x, y = T.dev_f32(noisy), T.dev_f32(clean)
        d.loss_grad(x, y, want_loss=False)
        once = d.grads().copy()
        d.loss_grad(x, y, want_loss=False, accumulate=True)
        twice = d.grads()
    assert np.any(once)
    assert np.array_equal(twice, 2 * once)


@pytest.mark.parametrize("shape,co,skip,relu,f32,shift", [
    ((3, 5, 7), 8, False, True, False, 0),     # less than a tile, a quarter of the channels
    ((5, 9, 17), 40, True, True, False, 0),    # one voxel past a tile, skip
    ((4, 4, 16), 64, False, False, True, 0),   # exactly a tile, FP32
    ((6, 7, 33), 100, True, True, True, 0),    # channels in fours
    ((4, 5, 20), 33, True, False, False, 0),
    ((4, 5, 20), 32, True, True, False, 3),    # operands off 16-byte alignment
])
def test_one_channel_layer_edges(shape, co, skip, relu, f32, shift):
    """3x3x3 layers of one input channel against the oracle on BF16 operands:
    FP32 sums of 27 products (1e-5 of the sum of their sizes), then one BF16
    rounding (2^-8) unless the output is FP32."""
    import test_gpu_nn as T
    t = T.torch()
    say("[gpu] one channel", shape, co, skip, relu, f32, shift)
    x, w, b = T.layer_case("conv3", shape, 1, co, 71)
    wq = T.O.bf16(w)
    sk = T.O.bf16(np.random.default_rng(72).standard_normal(shape + (co,))) if skip else None

    def placed(a, dtype):
        buf = t.zeros(a.size + shift, dtype=dtype, device="cuda")
        v = buf[shift:].view(a.shape)
        v.copy_(t.from_numpy(np.ascontiguousarray(a)))
        return v

    y = placed(np.zeros(shape + (co,), np.float32), t.float32 if f32 else t.bfloat16)
    T.nn.mcx_nn_layer_forward(T.nn.MCX_NN_CONV3, shape, 1, co, placed(x, t.bfloat16), T.dev_f32(w),
                              T.dev_f32(b), y=y, y_f32=f32, relu=relu,
                              skip=None if sk is None else placed(sk, t.bfloat16))
    ref = T.FWD["conv3"](x, wq, b)
    size = T.FWD["conv3"](np.abs(x), np.abs(wq), np.abs(b))
    if skip:
        ref, size = ref + sk, size + np.abs(sk)
    if relu:
        ref = np.maximum(ref, 0)
    got = y.float().cpu().numpy()
    lim = 1e-5 * size + (0 if f32 else 2.0 ** -8 * np.abs(ref))
    assert np.all(np.abs(got - ref) <= lim + 1e-30)


@pytest.mark.parametrize("shape,ci,co,skip,f32,shift", [
    ((5, 6, 7), 64, 40, True, False, 0),       # remainders of tiles and channels
    ((16, 36, 40), 96, 64, True, False, 0),    # deep tiles
    ((30, 64, 66), 64, 72, False, True, 0),    # deep tiles with padding, more tiles than workgroups
    ((20, 68, 72), 64, 64, False, False, 0),   # two slices, more tiles than workgroups
    ((9, 40, 44), 64, 24, True, False, 0),     # 32-channel tiles
    ((9, 10, 11), 64, 16, False, True, 0),     # four channels a lane
    ((9, 10, 11), 64, 12, True, False, 0),     # channels not in eights
    ((5, 6, 7), 64, 64, True, False, 3),       # operands off 16-byte alignment
    ((33, 40, 36), 32, 32, False, False, 0),   # weights in registers, remainders
])
def test_3x3x3_layer_edges(shape, ci, co, skip, f32, shift):
    """3x3x3 layers at the edges of their tilings against the oracle on BF16
    operands: FP32 sums (1e-5 of the sum of the products' sizes), then one BF16
    rounding (2^-8) unless the output is FP32."""
    import test_gpu_nn as T
    t = T.torch()
    say("[gpu] 3x3x3", shape, ci, co, skip, f32, shift)
    x, w, b = T.layer_case("conv3", shape, ci, co, 81)
    wq = T.O.bf16(w)
    sk = T.O.bf16(np.random.default_rng(82).standard_normal(shape + (co,))) if skip else None

    def placed(a, dtype):
        buf = t.zeros(a.size + shift, dtype=dtype, device="cuda")
        v = buf[shift:].view(a.shape)
        v.copy_(t.from_numpy(np.ascontiguousarray(a)))
        return v

    y = placed(np.zeros(shape + (co,), np.float32), t.float32 if f32 else t.bfloat16)
    T.nn.mcx_nn_layer_forward(T.nn.MCX_NN_CONV3, shape, ci, co, placed(x, t.bfloat16),
                              T.dev_f32(w), T.dev_f32(b), y=y, y_f32=f32, relu=True,
                              skip=None if sk is None else placed(sk, t.bfloat16))
    ref = T.FWD["conv3"](x, wq, b)
    size = T.FWD["conv3"](np.abs(x), np.abs(wq), np.abs(b))
    if skip:
        ref, size = ref + sk, size + np.abs(sk)
    ref = np.maximum(ref, 0)
    got = y.float().cpu().numpy()
    lim = 1e-5 * size + (0 if f32 else 2.0 ** -8 * np.abs(ref))
    assert np.all(np.abs(got - ref) <= lim + 1e-30)


@pytest.mark.parametrize("shape,ci,co", [((4, 4, 4), 8, 8), ((5, 6, 7), 16, 20), ((9, 4, 5), 24, 40),
                                         ((6, 5, 13), 40, 72), ((7, 8, 9), 56, 33),
                                         ((12, 14, 10), 48, 16)])
def test_few_channels_in_eights(shape, ci, co):
    """3x3x3 layers of 8 to 56 channels in eights, forward and the gradients
    (the input gradient gathers co channels), against the oracle."""
    say("[gpu] eights", shape, ci, co)
    layer_forward_backward("conv3", shape, ci, co, 91)
    layer_forward_backward("conv3", shape, 8 * (co // 8), ci, 92)
