"""The work whose speed is measured: calls of the framework's public entry
points over the sizes its users run.

Three families, each from its smallest calls to its largest: photon
transport (one simulation, the head phantom, many simulations in one
launch) with the map and the detector data read out; the post-processing of
detector records; and the denoiser (whole networks, a training step, single
layers forward and backward).  `listed` names the cases, `draw` gives
others of the same ranges, `prepare` makes what a program holds before the
call, `run` is one pass, `work` what a pass cannot do without, and `exact`
the outputs in 64 bits where they have such a value.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1711_03244_amd import mcx, nn
from paper_1711_03244_amd import workloads as W

LAYER_KINDS = {"conv3": nn.MCX_NN_CONV3, "down": nn.MCX_NN_DOWN, "up": nn.MCX_NN_UP}


def listed() -> list:
    return [
        # the smallest simulation worth a call: 1e4 photons of the paper's
        # homogeneous cube, where launches and the longest photon count
        {"name": "cube60_1e4", "kind": "transport", "domain": "cube", "side": 60, "ngates": 1,
         "photons": 10_000, "shape": "default"},
        # a quick look at the paper's heterogeneous benchmark: 50 gates,
        # Fresnel boundaries, four detectors, untuned
        {"name": "sphere60_1e6", "kind": "transport", "domain": "sphere", "side": 60,
         "ngates": 50, "photons": 1_000_000, "shape": "default"},
        # the same benchmark as a production run: large, with the launch
        # shape and census-shaped window a tuned program keeps
        {"name": "sphere60_3e7", "kind": "transport", "domain": "sphere", "side": 60,
         "ngates": 50, "photons": 30_000_000, "shape": "tuned"},
        # an atlas-sized head of five tissues, 7.1 M voxels and 10 gates
        {"name": "head_1e7", "kind": "transport", "domain": "head", "side": 0, "ngates": 10,
         "photons": 10_000_000, "shape": "default"},
        # independent cubes of 32 to 128 voxels a side in one launch (a
        # tenth of the batched workload's simulations and photons)
        {"name": "batch_24", "kind": "batch", "sims": 24, "scale": 0.1},
        # reflectance, time-resolved reflectance and absorption reweighting
        # of the benchmark's detected photons
        {"name": "detpost_250k", "kind": "detpost", "records": 250_000, "ndet": 4, "npath": 2,
         "ngates": 50, "reweight": True, "noalloc": False},
        # inference as the trained denoiser is evaluated: 64^3, averaged
        # over the eight symmetries
        {"name": "denoise_64_sym8", "kind": "denoise", "levels": 4, "width": 32, "nx": 64,
         "ny": 64, "nz": 64, "nsym": 8},
        # a small, ragged network: launches count
        {"name": "denoise_24_small", "kind": "denoise", "levels": 3, "width": 8, "nx": 24,
         "ny": 20, "nz": 28, "nsym": 1},
        # one optimiser step as the denoiser is trained: the gradients of
        # four 64^3 volumes, clipped, and Adam
        {"name": "train_64_b4", "kind": "train", "levels": 4, "width": 32, "nx": 64, "ny": 64,
         "nz": 64, "volumes": 4},
        # single layers, as a program with another graph calls them: a
        # ragged 3x3x3 convolution of the middle resolution,
        {"name": "conv3_fwd_30", "kind": "layer_fwd", "layer": "conv3", "nx": 30, "ny": 34,
         "nz": 28, "cin": 64, "cout": 64, "f32": False, "skip": False},
        # the gradients of a full-resolution one,
        {"name": "conv3_bwd_64", "kind": "layer_bwd", "layer": "conv3", "nx": 64, "ny": 64,
         "nz": 64, "cin": 32, "cout": 32},
        # and of a stride-2 transposed one
        {"name": "up_bwd_32", "kind": "layer_bwd", "layer": "up", "nx": 32, "ny": 32, "nz": 32,
         "cin": 64, "cout": 32},
    ]


def _log_int(rng, lo, hi) -> int:
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng) -> dict:
    kind = rng.choice(["transport", "transport", "head", "batch", "detpost", "denoise", "train",
                       "layer_fwd", "layer_fwd", "layer_bwd", "layer_bwd"])
    if kind == "transport":
        return {"kind": kind, "domain": rng.choice(["cube", "sphere"]),
                "side": rng.randint(24, 72), "ngates": rng.choice([1, 5, 10, 25, 50]),
                "photons": _log_int(rng, 1e4, 1e7), "shape": rng.choice(["default", "tuned"])}
    if kind == "head":
        return {"kind": "transport", "domain": "head", "side": 0, "ngates": 10,
                "photons": _log_int(rng, 1e5, 1e7), "shape": "default"}
    if kind == "batch":
        return {"kind": kind, "sims": rng.randint(3, 24),
                "scale": round(math.exp(rng.uniform(math.log(0.005), math.log(0.1))), 4)}
    if kind == "detpost":
        return {"kind": kind, "records": _log_int(rng, 1e3, 1e6), "ndet": rng.randint(1, 24),
                "npath": rng.randint(1, 5), "ngates": rng.randint(1, 100),
                "reweight": rng.random() < 0.7, "noalloc": rng.random() < 0.5}
    if kind in ("denoise", "train"):
        levels = rng.randint(2, 4)
        f = 2 ** (levels - 1)
        nx, ny, nz = (f * rng.randint(2, 64 // f) for _ in range(3))
        d = {"kind": kind, "levels": levels, "width": rng.choice([8, 16, 32]), "nx": nx,
             "ny": ny, "nz": nz}
        if kind == "train":
            d["volumes"] = rng.randint(1, 4)
        else:
            d["nsym"] = rng.choice([1, 2, 4, 8] if nx == ny else [1, 2, 4])
        return d
    layer = rng.choice(["conv3", "conv3", "down", "up"])
    hi = 32 if layer == "up" else 64
    nx, ny, nz = (_log_int(rng, 6, hi) for _ in range(3))
    if layer == "down":
        nx, ny, nz = (n + n % 2 for n in (nx, ny, nz))
    channels = [1, 8, 16, 24, 32, 40, 64, 96, 128, 256]
    cin, cout = rng.choice(channels[1:] if layer != "conv3" else channels), rng.choice(channels)
    while cin * cout * nx * ny * nz > 64 * 64 * 32 ** 3:  # the full-resolution layers' work
        if cin >= cout:
            cin = max(1, cin // 2)
        else:
            cout = max(1, cout // 2)
    d = {"kind": kind, "layer": layer, "nx": nx, "ny": ny, "nz": nz, "cin": cin, "cout": cout}
    if kind == "layer_fwd":
        d["f32"] = rng.random() < 0.3
        d["skip"] = rng.random() < 0.3
    return d


# --------------------------------------------------------------- transport


def _problem(case):
    if case["domain"] == "head":
        return W.head_phantom()
    if case["domain"] == "cube":
        return W.cube_homogeneous(case["side"]).replace(ngates=case["ngates"],
                                                        dt=5.0 / case["ngates"])
    return W.cube_sphere(case["side"], ngates=case["ngates"], dt=5.0 / case["ngates"])


def _prepare_transport(case, seed):
    p = _problem(case)
    sim = mcx.Simulation(p)
    if case["shape"] == "tuned":  # what autotune picks for the benchmark at full size
        sim.set_launch(1024, 64, 32768)
        sim.shape_window(200_000, 7, 32768)
    out = torch.empty(p.tally_shape, dtype=torch.float32, device="cuda")
    return {"sim": sim, "n": case["photons"], "seed": 1 + seed, "out": out, "ndet": p.ndet}


COUNTS = ("launched", "escaped", "timeout", "rr_dead", "scatters", "face_events", "detected")


def _run_transport(s):
    sim = s["sim"]
    sim.run(s["n"], s["seed"])
    phi = mcx.mcx_fluence_device(sim.ctx, mcx.MCX_FLUENCE_RATE, s["out"])
    st = sim.stats()
    r = {"map": phi, "absorbed": st["absorbed_grid"],
         "counts": np.array([st[k] for k in COUNTS], np.int64)}
    if s["ndet"]:
        r["reflectance"] = sim.detected_process()[0]
    return r


def _prepare_batch(case, seed):
    items = W.batch_workload(nsims=case["sims"], scale=case["scale"])
    b = mcx.Batch([it.problem for it in items])
    return {"batch": b, "n": [it.nphoton for it in items],
            "seed": [it.seed + 1009 * seed for it in items]}


def _run_batch(s):
    b = s["batch"]
    b.run(s["n"], s["seed"])
    maps, absorbed, counts = [], [], []
    for i in range(len(b)):
        maps.append(b.fluence(i))
        st = b.stats(i)
        absorbed.append(st["absorbed_grid"])
        counts.append([st[k] for k in COUNTS])
    return {"maps": maps, "absorbed": np.array(absorbed), "counts": np.array(counts, np.int64)}


# --------------------------------------------------------- post-processing


def _records(case, seed):
    """Detector records as a run leaves them: detectors of unequal share,
    weights below 1, log-normal exit times, pathlengths that add up to the
    path the time allows."""
    g = np.random.default_rng(seed)
    n, nd, npath = case["records"], case["ndet"], case["npath"]
    share = g.random(nd) + 0.2
    det = g.choice(nd, size=n, p=share / share.sum())
    t = np.minimum(np.exp(g.normal(-1.2, 0.7, n)), 4.999)
    parts = g.random((n, npath)) + 1e-3
    length = (t * 299.792458 / 1.37)[:, None] * parts / parts.sum(1, keepdims=True)
    w = np.exp(-0.005 * length.sum(1))
    rows = np.concatenate([det[:, None], np.floor(t * 200)[:, None], w[:, None], t[:, None],
                           length], axis=1)
    dmua = g.uniform(-0.002, 0.01, npath)
    return rows.astype(np.float32), dmua.astype(np.float32)


def _prepare_detpost(case, seed):
    rows, dmua = _records(case, seed)
    spec = {"ndet": case["ndet"], "npath": case["npath"], "t0": 0.0, "dt": 5.0 / case["ngates"],
            "ngates": case["ngates"], "nphoton": 100_000_000}
    dev = torch.device("cuda")
    return {"rec": torch.as_tensor(rows, device=dev), "spec": spec,
            "dmua": torch.as_tensor(dmua, device=dev) if case["reweight"] else None,
            "out": torch.empty((case["ndet"], 2 + case["ngates"]), dtype=torch.float64, device=dev),
            "weight": torch.empty(case["records"], dtype=torch.float64, device=dev),
            "noalloc": case["noalloc"]}


def _run_detpost(s):
    out, weight = mcx.mcx_detpost_device(s["rec"], s["spec"], dmua=s["dmua"], out=s["out"],
                                         weight=s["weight"], noalloc=s["noalloc"],
                                         stream=torch.cuda.current_stream())
    return {"out": out, "weight": weight}


def _exact_detpost(case, seed):
    rows, dmua = _records(case, seed)
    r = rows.astype(np.float64)
    w = r[:, 2]
    if case["reweight"]:
        w = w * np.exp(-(r[:, 4:] @ dmua.astype(np.float64)))
    dt = float(np.float32(5.0 / case["ngates"]))
    gate = np.clip(np.floor(r[:, 3] / dt), 0, case["ngates"] - 1).astype(np.int64)
    d = r[:, 0].astype(np.int64)
    out = np.zeros((case["ndet"], 2 + case["ngates"]))
    np.add.at(out, (d, 0), 1.0)
    np.add.at(out, (d, 1), w / 1e8)
    np.add.at(out, (d, 2 + gate), w / (1e8 * dt))
    return {"out": out, "weight": w}


# ---------------------------------------------------------------- denoiser


def _channels(case):
    return tuple(case["width"] * 2 ** i for i in range(case["levels"]))


def _net_params(case, seed):
    """(w, b) per layer; weights that BF16 holds exactly, as a trained
    checkpoint has them."""
    ws = W.denoiser_weights(_channels(case), seed=1 + seed, zero_output=False, bias_scale=0.02)
    out = []
    for i, (w, b) in enumerate(ws):
        if i == len(ws) - 1:
            w = 0.1 * w  # a residual: small against the map
        out.append((torch.as_tensor(w).to(torch.bfloat16).to(torch.float32).numpy(),
                    b.astype(np.float32)))
    return out


def _maps(case, seed, count):
    """Pairs of (noisy, clean) fluence maps per launched photon: a beam's
    diffuse fall-off through random inclusions, and what a run of few photons
    sees of it (counting noise, empty voxels far from the beam)."""
    g = np.random.default_rng([seed, 77])
    nz, ny, nx = case["nz"], case["ny"], case["nx"]
    z, y, x = np.meshgrid(np.arange(nz) + 0.5, np.arange(ny) + 0.5, np.arange(nx) + 0.5,
                          indexing="ij")
    pairs = []
    for _ in range(count):
        r = np.sqrt((x - nx / 2) ** 2 + (y - ny / 2) ** 2 + z ** 2)
        mu = g.uniform(0.1, 0.35)
        logphi = -mu * r - np.log(r + 1.0) - 2.0
        for _ in range(int(g.integers(1, 5))):
            c = [g.uniform(0, n) for n in (nx, ny, nz)]
            rad = g.uniform(0.1, 0.3) * min(nx, ny, nz)
            inside = (x - c[0]) ** 2 + (y - c[1]) ** 2 + (z - c[2]) ** 2 < rad ** 2
            logphi = logphi + g.uniform(-1.0, 0.5) * inside
        clean = np.exp(logphi)
        lam = np.maximum(clean * 1e6, 1e-6)
        noisy = g.poisson(np.minimum(lam, 1e6)) / 1e6
        pairs.append((noisy.astype(np.float32), clean.astype(np.float32)))
    return pairs


def _net(case, seed):
    den = nn.Denoiser(_channels(case), (case["nz"], case["ny"], case["nx"]))
    den.set_params(_net_params(case, seed))
    return den


def _prepare_denoise(case, seed):
    x = torch.as_tensor(_maps(case, seed, 1)[0][0]).cuda()
    return {"den": _net(case, seed), "x": x, "phi": torch.empty_like(x),
            "u": torch.empty_like(x), "nsym": case["nsym"]}


def _run_denoise(s):
    s["den"].forward(s["x"], phi_out=s["phi"], u_out=s["u"], symmetries=s["nsym"])
    return {"phi": s["phi"], "u": s["u"]}


def _prepare_train(case, seed):
    pairs = [(torch.as_tensor(a).cuda(), torch.as_tensor(b).cuda())
             for a, b in _maps(case, seed, case["volumes"])]
    return {"den": _net(case, seed), "pairs": pairs}


def _run_train(s):
    # the last steps of a decayed schedule: a rate that leaves the weights
    # where they are, so that every pass computes the same gradients
    den, n = s["den"], len(s["pairs"])
    for b, (x, y) in enumerate(s["pairs"]):
        den.loss_grad(x, y, want_loss=False, accumulate=b > 0)
    den.adam(1e-9, 1.0 / n, 0.1)
    return den.grads()


# ------------------------------------------------- the denoiser in 64 bits


def _to_u(phi):
    return (torch.log(torch.clamp(phi, min=float(np.float32(1e-12)))) + 16.0) / 4.0


def _layer64(kind, x, w, b):
    """x (z, y, x, cin), w (taps, cin, cout): the layer by its definition."""
    nz, ny, nx, _ = x.shape
    if kind == "conv3":
        p = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1, 1, 1))
        y = sum(p[a:a + nz, c:c + ny, e:e + nx] @ w[9 * a + 3 * c + e]
                for a in range(3) for c in range(3) for e in range(3))
    elif kind == "down":
        y = sum(x[t >> 2::2, (t >> 1) & 1::2, t & 1::2] @ w[t] for t in range(8))
    else:
        y = torch.stack([x @ w[t] for t in range(8)])
        y = y.reshape(2, 2, 2, nz, ny, nx, -1).permute(3, 0, 4, 1, 5, 2, 6)
        y = y.reshape(2 * nz, 2 * ny, 2 * nx, -1)
    return y if b is None else y + b


def _net64(case, params, u):
    """The network's output in u space, layer by layer, without rounding."""
    shapes = W.denoiser_layer_shapes(_channels(case))
    x, skips = u[..., None], []
    levels, level, last = case["levels"], 0, len(shapes) - 1
    for i, (kind, _, _, _) in enumerate(shapes):
        w, b = params[i]
        y = _layer64(kind, x, w, b)
        if kind == "up":
            level -= 1
            y = y + skips[level]
        elif kind == "down":
            level += 1
        x = y if i == last else torch.relu(y)
        if kind == "conv3" and i < 2 * levels and i % 2 == 1:
            skips.append(x)
    return u + x[..., 0]


def _params64(case, seed):
    return [(torch.as_tensor(w).double().cuda(), torch.as_tensor(b).double().cuda())
            for w, b in _net_params(case, seed)]


def _mirror(x, op):
    if op & 1:
        x = torch.flip(x, (2,))
    if op & 2:
        x = torch.flip(x, (1,))
    return x.transpose(1, 2) if op & 4 else x


def _exact_denoise(case, seed):
    params = _params64(case, seed)
    phi = torch.as_tensor(_maps(case, seed, 1)[0][0]).double().cuda()
    acc = 0.0
    for op in range(case["nsym"]):
        out = _net64(case, params, _to_u(_mirror(phi, op)))
        inv = (4 | ((op & 1) << 1) | ((op & 2) >> 1)) if op & 4 else op
        acc = acc + _mirror(out, inv)
    u = acc / case["nsym"]
    return {"phi": torch.exp(u * 4.0 - 16.0).cpu(), "u": u.cpu()}


def _exact_train(case, seed):
    params = _params64(case, seed)
    flat = [t.requires_grad_() for wb in params for t in wb]
    total = None
    for a, b in _maps(case, seed, case["volumes"]):
        y = torch.as_tensor(b).double().cuda()
        out = _net64(case, params, _to_u(torch.as_tensor(a).double().cuda()))
        mask = y >= 1e-8 * y.max()
        loss = ((out - _to_u(y))[mask] ** 2).mean()
        grads = torch.autograd.grad(loss, flat)
        grads = torch.cat([g.reshape(-1) for g in grads])
        total = grads if total is None else total + grads
    return total.cpu()


# ------------------------------------------------------------ single layers


def _taps(layer):
    return 27 if layer == "conv3" else 8


def _out_shape(case):
    s = (case["nz"], case["ny"], case["nx"])
    if case["layer"] == "down":
        return tuple(n // 2 for n in s)
    return tuple(2 * n for n in s) if case["layer"] == "up" else s


def _layer_inputs(case, seed):
    """Activations behind a ReLU, He-scaled weights, gradients behind a mask."""
    g = torch.Generator().manual_seed(1000 + seed)
    cin, cout = case["cin"], case["cout"]
    shape, out = (case["nz"], case["ny"], case["nx"]), _out_shape(case)
    taps = _taps(case["layer"])
    bf = lambda t: t.to(torch.bfloat16)  # noqa: E731
    d = {"x": bf(torch.relu(torch.randn(shape + (cin,), generator=g))),
         "w": bf(torch.randn((taps, cin, cout), generator=g)
                 * math.sqrt(2.0 / (taps * cin))).float()}
    if case["kind"] == "layer_fwd":
        d["b"] = 0.1 * torch.randn(cout, generator=g)
        if case["skip"]:
            d["skip"] = bf(torch.relu(torch.randn(out + (cout,), generator=g)))
    else:
        gy = 1e-3 * torch.randn(out + (cout,), generator=g)
        d["gy"] = bf(gy * (torch.rand(out + (cout,), generator=g) < 0.5))
    return d


def _prepare_layer(case, seed):
    s = {k: v.cuda() for k, v in _layer_inputs(case, seed).items()}
    s.update(case=dict(case))
    cin, cout = case["cin"], case["cout"]
    if case["kind"] == "layer_fwd":
        s["y"] = torch.empty(_out_shape(case) + (cout,), device="cuda",
                             dtype=torch.float32 if case["f32"] else torch.bfloat16)
    else:
        s["gx"] = torch.empty((case["nz"], case["ny"], case["nx"], cin), device="cuda")
        s["gw"] = torch.empty((_taps(case["layer"]), cin, cout), device="cuda")
        s["gb"] = torch.empty(cout, device="cuda")
    return s


def _run_layer(s):
    c = s["case"]
    args = (LAYER_KINDS[c["layer"]], (c["nz"], c["ny"], c["nx"]), c["cin"], c["cout"])
    if c["kind"] == "layer_fwd":
        return nn.mcx_nn_layer_forward(*args, s["x"], s["w"], s["b"], s.get("skip"), relu=True,
                                       y=s["y"], y_f32=c["f32"])
    nn.mcx_nn_layer_backward(*args, s["x"], s["w"], s["gy"], s["gx"], s["gw"], s["gb"])
    return {"gx": s["gx"], "gw": s["gw"], "gb": s["gb"]}


def _exact_layer(case, seed):
    d = {k: v.double().cuda() for k, v in _layer_inputs(case, seed).items()}
    if case["kind"] == "layer_fwd":
        y = _layer64(case["layer"], d["x"], d["w"], d["b"])
        return torch.relu(y + d["skip"] if case["skip"] else y).cpu()
    x, w = d["x"].requires_grad_(), d["w"].requires_grad_()
    gx, gw = torch.autograd.grad(_layer64(case["layer"], x, w, None), (x, w), d["gy"])
    return {"gx": gx.cpu(), "gw": gw.cpu(), "gb": d["gy"].sum((0, 1, 2)).cpu()}


# -------------------------------------------------------------- the contract


def prepare(case, seed):
    kind = case["kind"]
    if kind == "transport":
        return {"go": _run_transport, **_prepare_transport(case, seed)}
    if kind == "batch":
        return {"go": _run_batch, **_prepare_batch(case, seed)}
    if kind == "detpost":
        return {"go": _run_detpost, **_prepare_detpost(case, seed)}
    if kind == "denoise":
        return {"go": _run_denoise, **_prepare_denoise(case, seed)}
    if kind == "train":
        return {"go": _run_train, **_prepare_train(case, seed)}
    return {"go": _run_layer, **_prepare_layer(case, seed)}


def run(state):
    return state["go"](state)


def exact(case, seed):
    kind = case["kind"]
    if kind == "detpost":
        return _exact_detpost(case, seed)
    if kind == "denoise":
        return _exact_denoise(case, seed)
    if kind == "train":
        return _exact_train(case, seed)
    if kind in ("layer_fwd", "layer_bwd"):
        return _exact_layer(case, seed)
    return None  # a random walk's map has no closed value


# Segments per photon of the workloads (a 60-voxel cube, the head, the mean
# of the batched cubes) and the operations of a segment: free path, three
# face distances, the deposit, and a scattering or a crossing.
SEGMENTS = {"cube": 196, "sphere": 378, "head": 921, "batch": 667}
SEGMENT_OPS = 130


def _layer_flops(kind, cin, cout, in_vox):
    if kind == "conv3":
        return 2 * 27 * cin * cout * in_vox
    return 2 * 8 * cin * cout * (in_vox // 8 if kind == "down" else in_vox)


def _net_flops(case):
    vox, total = case["nx"] * case["ny"] * case["nz"], 0
    for kind, _, ci, co in W.denoiser_layer_shapes(_channels(case)):
        total += _layer_flops(kind, ci, co, vox)
        vox = vox // 8 if kind == "down" else vox * 8 if kind == "up" else vox
    return total


def _net_nparam(case):
    return sum(t * ci * co + co for _, t, ci, co in W.denoiser_layer_shapes(_channels(case)))


def work(case):
    kind = case["kind"]
    if kind == "transport":
        nvox = int(np.prod(W.HEAD_SHAPE)) if case["domain"] == "head" else case["side"] ** 3
        scale = case["side"] / 60 if case["side"] else 1.0
        return {"bytes": nvox * (1 + 4 * case["ngates"]),
                "flops": case["photons"] * SEGMENTS[case["domain"]] * scale * SEGMENT_OPS}
    if kind == "batch":
        vox = case["sims"] * sum(s ** 3 for s in W.BATCH_SIDES) / len(W.BATCH_SIDES)
        lo, hi = W.BATCH_PHOTONS
        n = case["sims"] * case["scale"] * (hi - lo) / math.log(hi / lo)
        return {"bytes": vox * 5, "flops": n * SEGMENTS["batch"] * SEGMENT_OPS}
    if kind == "detpost":
        n = case["records"]
        return {"bytes": n * (4 * (4 + case["npath"]) + 8), "flops": n * (2 * case["npath"] + 20)}
    if kind in ("denoise", "train"):
        vox = case["nx"] * case["ny"] * case["nz"]
        if kind == "denoise":
            return {"bytes": 12 * vox + 2 * _net_nparam(case),
                    "flops": case["nsym"] * _net_flops(case)}
        return {"bytes": 8 * vox * case["volumes"] + 28 * _net_nparam(case),
                "flops": 3 * case["volumes"] * _net_flops(case)}
    vox_in, vox_out = case["nx"] * case["ny"] * case["nz"], int(np.prod(_out_shape(case)))
    cin, cout = case["cin"], case["cout"]
    flops = _layer_flops(case["layer"], cin, cout, vox_in)
    weights = _taps(case["layer"]) * cin * cout
    if kind == "layer_fwd":
        return {"bytes": 2 * vox_in * cin + 4 * weights + vox_out * cout
                * ((4 if case["f32"] else 2) + (2 if case["skip"] else 0)), "flops": flops}
    return {"bytes": 6 * vox_in * cin + 2 * vox_out * cout + 8 * weights, "flops": 2 * flops}
