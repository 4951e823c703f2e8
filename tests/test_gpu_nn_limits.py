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


def placed(a, dtype, shift):
    """`a` in device memory, `shift` elements past a 16-byte boundary"""
    t = T.torch()
    buf = t.zeros(a.size + shift, dtype=dtype, device="cuda")
    v = buf[shift:].view(a.shape)
    v.copy_(t.from_numpy(np.ascontiguousarray(a, np.float32)))
    return v


@pytest.mark.parametrize("co,f32,shift", [(32, False, 1), (32, True, 1), (16, False, 3),
                                          (40, False, 4), (8, True, 2)])
def test_resident_grids_with_outputs_off_alignment(co, f32, shift):
    """3x3x3 layers of 32 channels on a grid of 1024 tiles whose output alone
    is off 16-byte alignment: the same values as an aligned output (FP32 sums
    in another order: 1e-5 of the sum of the products' sizes, and one BF16
    rounding, 2^-7, where the output is BF16)."""
    t = T.torch()
    shape = (33, 64, 62)
    say("[gpu] output off alignment", co, f32, shift)
    x, w, b = T.layer_case("conv3", shape, 32, co, 5)
    dt = t.float32 if f32 else t.bfloat16
    xd, wd, bd = T.dev_bf16(x), T.dev_f32(w), T.dev_f32(b)
    ys = []
    for sh in (0, shift):
        y = placed(np.full(shape + (co,), 7.0, np.float32), dt, sh)
        T.nn.mcx_nn_layer_forward(T.nn.MCX_NN_CONV3, shape, 32, co, xd, wd, bd, relu=False, y=y,
                                  y_f32=f32)
        ys.append(T.host(y))
    size = t.nn.functional.conv3d(
        t.as_tensor(np.abs(x)).cuda().permute(3, 0, 1, 2)[None].float(),
        t.as_tensor(np.abs(w)).cuda().reshape(3, 3, 3, 32, co).permute(4, 3, 0, 1, 2).float(),
        padding=1)[0].permute(1, 2, 3, 0)
    lim = 1e-5 * T.host(size) + (0 if f32 else 2.0 ** -7 * np.abs(ys[0])) + 1e-6
    assert np.all(np.abs(ys[0] - ys[1]) <= lim)


@pytest.mark.parametrize("xs,gs", [(3, 0), (0, 3), (1, 1)])
@pytest.mark.parametrize("kind,shape,ci,co", [("conv3", (9, 8, 7), 32, 32), ("conv3", (6, 5, 7), 64, 12),
                                              ("conv3", (6, 5, 7), 24, 8), ("down", (4, 6, 4), 32, 40),
                                              ("up", (3, 4, 5), 8, 32)])
def test_weight_gradients_of_operands_off_alignment(kind, shape, ci, co, xs, gs):
    """Weight gradients where the activations, the output gradients or both
    are off 16-byte alignment, against the oracle on BF16 operands: 1e-5 of the
    sum of the products' sizes."""
    t = T.torch()
    say("[gpu] operands off alignment", kind, shape, ci, co, xs, gs)
    x, w, _ = T.layer_case(kind, shape, ci, co, 51)
    gy = T.O.bf16(np.random.default_rng(52).normal(size=T.out_shape(kind, shape) + (co,)))
    ref = T.BWD[kind](x, T.O.bf16(w), gy)
    lim = T.BWD[kind](np.abs(x), np.abs(T.O.bf16(w)), np.abs(gy))
    gw = t.full(w.shape, float("nan"), device="cuda")
    gb = t.full((co,), float("nan"), device="cuda")
    T.nn.mcx_nn_layer_backward(T.KIND[kind], shape, ci, co, placed(x, t.bfloat16, xs), T.dev_f32(w),
                               placed(gy, t.bfloat16, gs), None, gw, gb)
    assert np.all(np.abs(T.host(gw) - ref[1]) <= 1e-5 * lim[1] + 1e-30)
    size = np.abs(gy).reshape(-1, co).sum(0)
    assert np.all(np.abs(T.host(gb) - ref[2]) <= 1e-5 * size + 1e-30)


def free_bytes():
    t = T.torch()
    t.cuda.synchronize()
    return t.cuda.mem_get_info()[0]


@pytest.mark.parametrize("shape,images", [((32, 32, 32), 8), ((32, 32, 48), 4)])
def test_images_take_memory_with_the_first_symmetric_call(shape, images):
    """The memory of images that share launches comes with the first call that
    averages over symmetries, for as many as the cross-section has (four where
    nx != ny), and not with every network."""
    t = T.torch()
    channels = (32, 64)
    nz, ny, nx = shape
    vox = nz * ny * nx
    # the layers' outputs: four at full resolution, three at half, one voxel wide
    # input and output
    image = vox * (2 * (32 * 4 + 64 * 3 / 8) + 6)
    _, flat = T.make_net(channels, shape, 31)
    noisy, clean = T.fluence_pair(shape, 32)
    x, y = T.dev_f32(noisy), T.dev_f32(clean)
    u, u1 = t.empty_like(x), t.empty_like(x)
    say("[gpu] memory of images", shape)
    with T.nn.Denoiser(channels, shape) as d:
        d.set_params(flat)
        d.forward(x, u_out=u)
        d.loss_grad(x, y, want_loss=False)
        before = free_bytes()
        d.forward(x, u_out=u, symmetries=2)
        held = before - free_bytes()
        d.forward(x, u_out=u1, symmetries=4)
        d.forward(x, u_out=u1, symmetries=2)
        assert before - free_bytes() == held  # once
    assert t.equal(u, u1)
    # allocations come in pages of 2 MiB, and a workspace of split sums with them
    assert (images - 0.5) * image < held < (images + 0.5) * image + (40 << 20)


def test_symmetric_call_captured_first():
    """A graph that holds a network's first call over symmetries: its images go
    one at a time, and every replay gives the bits of the images that share
    launches, also after an eager call took memory for those."""
    t = T.torch()
    channels, shape = (16, 32), (12, 16, 16)
    _, flat = T.make_net(channels, shape, 33)
    x = T.dev_f32(T.fluence_pair(shape, 34)[0])
    other = T.dev_f32(T.fluence_pair(shape, 35)[0])
    say("[gpu] symmetric call under capture")
    want = []
    with T.nn.Denoiser(channels, shape) as d:
        d.set_params(flat)
        for v in (x, other):
            u = t.empty_like(x)
            d.forward(v, u_out=u, symmetries=8)
            want.append(u)
    with T.nn.Denoiser(channels, shape) as d:
        d.set_params(flat)
        d.forward(x, u_out=t.empty_like(x))  # packs the weights
        t.cuda.synchronize()
        inp, out = x.clone(), t.empty_like(x)
        g = t.cuda.CUDAGraph()
        with t.cuda.graph(g):
            d.forward(inp, u_out=out, symmetries=8)
        for k in (0, 1, 0, 1):
            inp.copy_((x, other)[k])
            out.zero_()
            g.replay()
            t.cuda.synchronize()
            assert t.equal(out, want[k])
            eager = t.empty_like(x)
            d.forward(inp, u_out=eager, symmetries=8)
            t.cuda.synchronize()
            assert t.equal(eager, want[k])


@pytest.mark.parametrize("value", [np.inf, np.nan])
@pytest.mark.parametrize("kind,shape,ci,co", [
    ("conv3", (5, 6, 19), 1, 40),        # one channel
    ("conv3", (6, 5, 7), 8, 16), ("conv3", (5, 7, 6), 40, 24),   # few channels in eights
    ("conv3", (9, 10, 11), 64, 40),      # bricks
    ("conv3", (33, 64, 62), 32, 32),     # resident weights
    ("up", (3, 5, 6), 64, 24), ("down", (6, 4, 10), 32, 16)])
def test_outputs_of_activations_not_finite(kind, shape, ci, co, value):
    """One activation that is not finite: the outputs it is part of are not
    finite, all others keep the bits they have with a zero in its place."""
    t = T.torch()
    say("[gpu] not finite, forward", value, kind, shape, ci, co)
    x, w, b = T.layer_case(kind, shape, ci, co, 9)
    w = np.abs(w) + 0.01  # no product of infinity and zero
    at = (shape[0] - 2, shape[1] - 1, 1)
    out = T.out_shape(kind, shape) + (co,)
    ys = []
    for v in (0.0, value):
        x[at + (ci // 2,)] = v
        y = t.empty(out, device="cuda")
        T.nn.mcx_nn_layer_forward(T.KIND[kind], shape, ci, co, T.dev_bf16(x), T.dev_f32(w),
                                  T.dev_f32(b), relu=False, y=y, y_f32=True)
        ys.append(T.host(y))
    part = np.zeros(out, bool)
    if kind == "conv3":
        part[tuple(slice(max(k - 1, 0), k + 2) for k in at)] = True
    elif kind == "up":
        part[tuple(slice(2 * k, 2 * k + 2) for k in at)] = True
    else:
        part[tuple(k // 2 for k in at)] = True
    assert np.all(np.isfinite(ys[0]))
    assert np.array_equal(~np.isfinite(ys[1]), part)
    assert np.array_equal(ys[1][~part], ys[0][~part])


@pytest.mark.parametrize("value", [np.inf, np.nan])
@pytest.mark.parametrize("kind,shape,ci,co", [("down", (6, 10, 14), 24, 72), ("down", (2, 2, 2), 8, 8),
                                              ("up", (5, 3, 7), 72, 24), ("up", (1, 1, 1), 8, 8)])
def test_stride_2_weight_gradients_not_finite(kind, shape, ci, co, value):
    """The last voxel's activation of one channel is not finite: so are that
    channel's weight gradients, of the one tap that reads it in a down layer
    and of all in an up layer, and no other ones."""
    t = T.torch()
    say("[gpu] not finite, stride 2", value, kind, shape, ci, co)
    rng = np.random.default_rng(8)
    x = T.O.bf16(np.abs(rng.normal(size=shape + (ci,))))
    gy = T.O.bf16(rng.uniform(0.5, 1.5, size=T.out_shape(kind, shape) + (co,)))
    x[-1, -1, -1, 3] = value
    gw = t.empty((8, ci, co), device="cuda")
    w = t.zeros((8, ci, co), device="cuda")
    T.nn.mcx_nn_layer_backward(T.KIND[kind], shape, ci, co, T.dev_bf16(x), w, T.dev_bf16(gy), None,
                               gw, None)
    part = np.zeros((8, ci, co), bool)
    part[7 if kind == "down" else slice(None), 3] = True
    assert np.array_equal(~np.isfinite(T.host(gw)), part)
