"""Workloads of the library's hot path, each timed as one pass through the public
entry points of ``paper_2412_09775_amd.api``.

``listed()`` names the workloads, ``draw(rng)`` gives another one of the same ranges;
``prepare`` makes what a program has in hand before the call (optics, data, workspaces),
``run`` is one pass, ``work`` what the pass cannot do without, and ``exact`` the same
outputs from plain FP64 torch.  Kinds:

* step     transfer-function synthesis + Tikhonov reconstruction of a 3D volume
* fwdadj   forward model d = H f + b and its backward (the adjoint) with a kept bank
* grad     differentiable 3D reconstruction: forward, then dL/dd and dL/dtheta
* midband  mid-band loss and its parameter gradient of a batch of defocus stacks
* restore  auto-tune and thin reconstruction of tiles of uneven shapes in one call
* cnn      forward, loss and gradient of the learned initialiser on one batch
* conv     one convolution layer of it: forward, input gradient, weight gradient
"""

import math

import numpy as np
import torch

DEV = "cuda"
FLUOR, LABELFREE, THIN, POL5, SECTORS9, VECTOR = range(6)
MODELS = {"fluor": FLUOR, "labelfree": LABELFREE, "pol5": POL5, "sectors9": SECTORS9, "vector4": VECTOR,
          "vector5": VECTOR}
CHANNELS = {"fluor": (1, 1), "labelfree": (1, 2), "pol5": (5, 4), "sectors9": (9, 1), "vector4": (4, 4),
            "vector5": (5, 4)}
VEC_PROPS = (0, 16, 8, 1)
SWING = 0.1
CNN_CHANNELS = (1, 32, 64, 128, 256)


# ---------------------------------------------------------------- the cases

def _step(name, model, layout, n, nz, ny, nx, dz, na_ill, na_det, edge=0.0, tilt=0.0, defocus=0.0):
    c = dict(kind="step", model=model, layout=layout, n=n, nz=nz, ny=ny, nx=nx, dz=dz, na_ill=na_ill,
             na_det=na_det, edge=edge, tilt=tilt, defocus=defocus)
    return dict(c, name=name) if name else c


def listed():
    return [
        # one small bead volume in a viewer or a serving loop: launches and host time count
        _step("fluor_32x64x64", "fluor", "full", 1, 32, 64, 64, 0.25, 0.0, 1.2),
        # the ordinary label-free volume, phase and absorption from one channel
        _step("labelfree_96x512x512", "labelfree", "band", 1, 96, 512, 512, 0.2, 0.5, 1.2),
        # the largest volume: five polarisation states to four properties
        _step("pol5_64x1024x1024", "pol5", "band", 1, 64, 1024, 1024, 0.25, 0.5, 0.75),
        # high-aperture birefringence: the vector bank of the five swing states
        _step("vector5_64x512x512", "vector5", "band", 1, 64, 512, 512, 0.25, 0.5, 0.75),
        # nine-aperture phase of a beating cell sheet
        _step("sectors9_48x512x512", "sectors9", "band", 1, 48, 512, 512, 0.2, 0.5, 1.2),
        # a crop as a user draws it: ragged sizes, tilted source, soft pupils, the full bank
        _step("labelfree_75x270x450", "labelfree", "full", 1, 75, 270, 450, 0.2, 0.5, 1.1, 1.76, 0.12, 0.3),
        # an iterative solver's inner step on two volumes: forward model and its adjoint
        dict(name="fwdadj_2x48x320x384", kind="fwdadj", model="labelfree", n=2, nz=48, ny=320, nx=384, dz=0.2,
             na_ill=0.5, na_det=1.1, edge=1.5, tilt=0.0, defocus=0.0),
        # tuning a 3D reconstruction through its own gradient
        dict(name="grad_48x256x256", kind="grad", model="labelfree", n=1, nz=48, ny=256, nx=256, dz=0.2,
             na_ill=0.5, na_det=1.1, edge=1.0, tilt=0.1, defocus=0.2),
        # one gradient evaluation of a plate's patches
        dict(name="midband_256x32x128x128", kind="midband", n=256, nz=32, ny=128, nx=128, edge=0.5),
        # a whole restoration: uneven tiles from learned starts, 20 iterations, reconstruction
        dict(name="restore_64tiles", kind="restore", n=64, iters=20, shapes=5001),
        # one gradient of the learned initialiser's training
        dict(name="cnn_64x32x64x64", kind="cnn", n=64, nz=32, ny=64, nx=64),
        # its third layer alone
        dict(name="conv_64x8x16x16_64to128", kind="conv", n=64, nz=8, ny=16, nx=16, cin=64, cout=128),
    ]


def _smooth(lo, hi, even):
    out = []
    for v in range(lo, hi + 1):
        m = v
        for p in (2, 3, 5):
            while m % p == 0:
                m //= p
        if m == 1 and not (even and v % 2):
            out.append(v)
    return out


def _size(rng, lo, hi, even=True):
    """A {2, 3, 5}-smooth size, spread over its logarithm."""
    want = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return min(_smooth(lo, hi, even), key=lambda v: abs(math.log(v / want)))


RESTORE_Z = (16, 24, 32, 48, 64)
RESTORE_YX = (128, 160, 192, 240, 256, 320, 384, 480, 512)


def draw(rng):
    kind = rng.choice(("step", "step", "step", "step", "fwdadj", "grad", "midband", "restore", "cnn", "conv"))
    if kind in ("step", "fwdadj", "grad"):
        model = rng.choice(tuple(CHANNELS)) if kind == "step" else "labelfree"
        if kind == "fwdadj":
            model = rng.choice(("fluor", "labelfree", "pol5"))
        cap = {"fluor": 3e7, "labelfree": 3e7, "pol5": 5e7, "sectors9": 1.3e7, "vector4": 1.5e7,
               "vector5": 1.5e7}[model]
        if kind == "grad":
            cap = 8e6
        while True:
            nz, ny, nx = _size(rng, 16, 96, False), _size(rng, 64, 1024), _size(rng, 64, 1024)
            n = rng.choice((1, 1, 1, 2, 3))
            if n * nz * ny * nx <= cap:
                break
        na_det = round(rng.uniform(0.7, 1.15), 3)
        soft = kind == "grad" or rng.random() < 0.5
        c = dict(kind=kind, model=model, n=n, nz=nz, ny=ny, nx=nx, dz=0.2,
                 na_ill=0.0 if model == "fluor" else round(rng.uniform(0.4, 0.6), 3), na_det=na_det,
                 edge=round(0.5 * max(ny, nx) / 128.0, 3) if soft else 0.0,
                 tilt=0.0 if model in ("fluor", "sectors9") else round(rng.choice((0.0, 1.0)) * rng.uniform(0.02, 0.2), 3),
                 defocus=round(rng.choice((0.0, 1.0)) * rng.uniform(-0.5, 0.5), 3))
        if kind == "step":
            c["layout"] = "full" if model == "fluor" or rng.random() < 0.3 else "band"
        return c
    if kind == "midband":
        while True:
            nz, ny, nx = _size(rng, 8, 64, False), _size(rng, 64, 512), _size(rng, 64, 512)
            n = int(round(math.exp(rng.uniform(0.0, math.log(256)))))
            if n * nz * ny * nx <= 1.3e8:
                return dict(kind=kind, n=n, nz=nz, ny=ny, nx=nx, edge=round(0.5 * max(ny, nx) / 128.0, 3))
    if kind == "restore":
        return dict(kind=kind, n=int(round(math.exp(rng.uniform(math.log(2), math.log(60))))),
                    iters=rng.randint(3, 20), shapes=rng.randrange(1 << 20))
    if kind == "cnn":
        return dict(kind=kind, n=rng.randint(3, 64), nz=rng.choice((16, 24, 32)), ny=rng.choice((48, 50, 64)),
                    nx=rng.choice((48, 50, 64)))
    i = rng.choice((1, 2, 3))
    f = 2 ** i
    return dict(kind="conv", n=rng.randint(3, 64), nz=32 // f, ny=rng.choice((48, 56, 64)) // f,
                nx=rng.choice((48, 56, 64)) // f, cin=CNN_CHANNELS[i], cout=CNN_CHANNELS[i + 1])


# ---------------------------------------------------------------- optics and inputs

def _optics(c, **kw):
    from paper_2412_09775_amd import api
    model = c.get("model")
    v = dict(model=THIN if model is None else MODELS[model], nz=c["nz"], ny=c["ny"], nx=c["nx"],
             dz=c.get("dz", 0.2), dy=0.1, dx=0.1, wavelength=0.52 if model == "fluor" else 0.532,
             na_ill=c.get("na_ill", 0.5), na_det=c.get("na_det", 1.15), n_medium=1.33,
             defocus=c.get("defocus", 0.0), tilt_zenith=c.get("tilt", 0.0), tilt_azimuth=0.0,
             edge_width=c.get("edge", 0.0), swing=SWING,
             vec_channels=1 if model == "vector5" else 0, vec_props=VEC_PROPS)
    v.update(kw)
    return api.Optics(**v)


def _patches(c):
    """Optics of the case's patches: a drift of defocus and aperture from patch to patch."""
    return [_optics(c, defocus=c["defocus"] + 0.1 * i, na_det=c["na_det"] * (1.0 - 0.02 * i))
            for i in range(c["n"])]


def _eta(c):
    """About 1e-3 of the bank's largest singular value squared (2 nz for an open label-free channel)."""
    if c["model"] == "fluor":
        return 1e-3
    return 1e-3 * (2.0 * c["nz"]) ** 2 * (0.2 if c["model"] in ("pol5", "vector5") else 1.0)


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _volume(shape, seed, noise):
    """Smooth random structures plus noise: (..., Z, Y, X)."""
    g = _gen(seed)
    lead, (Z, Y, X) = shape[:-3], shape[-3:]
    m = math.prod(lead)
    coarse = torch.randn((m, 1, max(Z // 4, 2), max(Y // 8, 2), max(X // 8, 2)), generator=g, device=DEV)
    x = torch.nn.functional.interpolate(coarse, size=(Z, Y, X), mode="trilinear").reshape(shape)
    return x.mul_(0.05).add_(torch.randn(shape, generator=g, device=DEV), alpha=noise)


def _beads(shape, seed):
    """Bright beads at random voxels, slightly blurred, plus noise."""
    n, _, Z, Y, X = shape
    rng = np.random.default_rng(seed)
    x = torch.zeros(shape, device=DEV)
    k = max(50, Z * Y * X // 5000)
    at = [torch.from_numpy(rng.integers(0, s, (n, k))).to(DEV) for s in (Z, Y, X)]
    amp = torch.from_numpy(rng.uniform(0.5, 1.0, (n, k)).astype(np.float32)).to(DEV)
    for i in range(n):
        x[i, 0][at[0][i], at[1][i], at[2][i]] = amp[i]
    x = torch.nn.functional.avg_pool3d(x, 3, 1, 1, count_include_pad=True) * 9
    return x.add_(torch.randn(shape, generator=_gen(seed), device=DEV), alpha=1e-3)


def _cells(n, ny, nx, seed):
    """Thin cells (n, 2, ny, nx): dome-shaped ellipses, phase U(0.1, 0.5), absorption U(0, 0.02)."""
    rng = np.random.default_rng(seed)
    k = max(1, round(20 * ny * nx / 128 ** 2))
    cast = lambda a: torch.from_numpy(np.asarray(a, dtype=np.float32)).to(DEV)  # noqa: E731
    cy, cx = cast(rng.uniform(0, ny, (n, k))), cast(rng.uniform(0, nx, (n, k)))
    ay, ax = cast(rng.uniform(8, 25, (n, k))), cast(rng.uniform(8, 25, (n, k)))
    ph, ab = cast(rng.uniform(0.1, 0.5, (n, k))), cast(rng.uniform(0.0, 0.02, (n, k)))
    y = torch.arange(ny, device=DEV, dtype=torch.float32)[:, None]
    x = torch.arange(nx, device=DEV, dtype=torch.float32)[None, :]
    out = torch.zeros((n, 2, ny, nx), device=DEV)
    for j in range(k):
        col = lambda a: a[:, j, None, None]  # noqa: E731
        dome = (1 - ((y - col(cy)) / col(ay)) ** 2 - ((x - col(cx)) / col(ax)) ** 2).clamp_(min=0).sqrt_()
        out[:, 0] += col(ph) * dome
        out[:, 1] += col(ab) * dome
    return out


def _dft(n, sign):
    k = np.arange(n)
    m = np.exp(sign * 2j * np.pi * (np.outer(k, k) % n) / n)
    return torch.from_numpy(m.astype(np.complex64)).to(DEV)


def _thin_stacks(nz, ny, nx, edge, theta, seed, noise=0.0317):
    """Defocus stacks (n, nz, ny, nx) of thin cells seen through the thin model at theta."""
    n = len(theta)
    cells = _cells(n, ny, nx, seed)
    fy, fx, iy, ix = _dft(ny, -1), _dft(nx, -1), _dft(ny, 1) / ny, _dft(nx, 1) / nx
    fwd = lambda v: fy @ (v @ fx)  # noqa: E731
    inv = lambda v: iy @ (v @ ix)  # noqa: E731
    g = _gen(seed)
    out = torch.empty((n, nz, ny, nx), device=DEV)
    step = max(1, int(2 ** 23 // (nz * ny * nx)))
    z = 0.2 * (torch.arange(nz, device=DEV, dtype=torch.float64) - (nz - 1) / 2)
    for i in range(0, n, step):
        th = torch.from_numpy(theta[i:i + step]).to(DEV)
        a, b, s = _arms(dict(nz=nz, ny=ny, nx=nx, edge=edge), th, z)
        c = inv(b.to(torch.complex64)) * inv(a.to(torch.complex64)).conj() * s.float()[:, None, None, None]
        obj = fwd(cells[i:i + step].to(torch.complex64))
        d = fwd((2 * c.real).to(torch.complex64)) * obj[:, :1] - fwd((2 * c.imag).to(torch.complex64)) * obj[:, 1:]
        out[i:i + step] = inv(d).real
    return out.add_(torch.randn(out.shape, generator=g, device=DEV), alpha=noise)


def _prior(n, seed):
    rng = np.random.default_rng(seed)
    return np.stack([rng.uniform(-2, 2, n), rng.uniform(1.0, 1.3, n) * 0.98,
                     rng.uniform(0.0, math.radians(30.0), n), np.zeros(n)], 1)


def _restore_shapes(c):
    rng = np.random.default_rng(c["shapes"])
    return [(int(rng.choice(RESTORE_Z)), int(rng.choice(RESTORE_YX)), int(rng.choice(RESTORE_YX)))
            for _ in range(c["n"])]


NU_C = (1.15 + 0.5) / 0.532


def _thin_eta(nz):
    """About 1e-2 of the thin bank's largest singular value squared."""
    return 0.05 * nz


def _linear_input(c, seed):
    C, P = CHANNELS[c["model"]]
    vol = (c["nz"], c["ny"], c["nx"])
    if c["kind"] == "fwdadj":
        if c["model"] == "fluor":
            return _beads((c["n"], P) + vol, seed)
        return _volume((c["n"], P) + vol, seed, 0.002)
    if c["model"] == "fluor":
        return _beads((c["n"], C) + vol, seed)
    return _volume((c["n"], C) + vol, seed, 0.01)


def _cnn_params(seed):
    rng = np.random.default_rng(seed)
    out = []
    for ci, co in zip(CNN_CHANNELS[:-1], CNN_CHANNELS[1:]):
        out += [rng.standard_normal(co * 27 * ci) * math.sqrt(2.0 / (27 * ci)), 0.02 * rng.standard_normal(co)]
    out += [rng.standard_normal(3 * 256) / 16.0, np.zeros(3)]
    return torch.from_numpy(np.concatenate(out).astype(np.float32)).to(DEV)


def _cnn_input(c, seed):
    theta = _prior(c["n"], seed + 1)
    x = _thin_stacks(c["nz"], c["ny"], c["nx"], 0.25, theta, seed)
    lo, hi = np.array([-2.0, 1.0, 0.0]), np.array([2.0, 1.3, math.radians(30.0)])
    t = 2.0 * (theta[:, :3] - lo) / (hi - lo) - 1.0
    return _cnn_params(seed), x, torch.from_numpy(t.astype(np.float32)).to(DEV)


def _conv_sizes(c):
    return (c["nz"] - 1) // 2 + 1, (c["ny"] - 1) // 2 + 1, (c["nx"] - 1) // 2 + 1


def _conv_input(c, seed):
    g = _gen(seed)
    x = torch.randn((c["n"], c["nz"], c["ny"], c["nx"], c["cin"]), generator=g, device=DEV)
    x = torch.nn.functional.gelu(x).to(torch.bfloat16)
    w = torch.randn((c["cout"], 27 * c["cin"]), generator=g, device=DEV) * math.sqrt(2.0 / (27 * c["cin"]))
    gz = torch.randn((c["n"], *_conv_sizes(c), c["cout"]), generator=g, device=DEV) * 1e-3
    return x, w.to(torch.bfloat16), gz.to(torch.bfloat16)


def prepare(case, seed):
    from paper_2412_09775_amd import api
    c = dict(case)
    s = {"case": c, "api": api}
    kind = c["kind"]
    if kind in ("step", "fwdadj"):
        s["optics"] = o = _patches(c)
        s["x"] = _linear_input(c, seed)
        s["eta"] = _eta(c)
        ops = ((api.OP_TRANSFER_FUNCTION, api.OP_RECONSTRUCT) if kind == "step" else
               (api.OP_TRANSFER_FUNCTION, api.OP_FORWARD, api.OP_ADJOINT))
        s["ws"] = torch.empty(max(api.workspace_size(o, op) for op in ops), dtype=torch.uint8, device=DEV)
        if kind == "step":
            dims = api.band_dims(o) if c["layout"] == "band" else api.bank_dims(o)
            s["tf"] = torch.empty(dims, dtype=torch.complex64, device=DEV)
        else:
            s["tf"] = api.transfer_function(o, device=DEV, ws=s["ws"])
            C = CHANNELS[c["model"]][0]
            s["b"] = torch.full((c["n"], C), 0.01, device=DEV)
            s["x"].requires_grad_(True)
            s["g"] = _volume((c["n"], C, c["nz"], c["ny"], c["nx"]), seed + 1, 0.01)
    elif kind == "grad":
        s["optics"] = o = _patches(c)
        s["eta"] = _eta(c)
        s["x"] = _linear_input(c, seed).requires_grad_(True)
        s["theta"] = torch.tensor([[p.defocus, p.na_det, p.tilt_zenith, p.tilt_azimuth] for p in o],
                                  dtype=torch.float64, requires_grad=True)
        P = CHANNELS[c["model"]][1]
        s["g"] = _volume((c["n"], P, c["nz"], c["ny"], c["nx"]), seed + 1, 0.01) * 1e-4
    elif kind == "midband":
        truth = _prior(c["n"], seed + 1)
        s["d"] = _thin_stacks(c["nz"], c["ny"], c["nx"], c["edge"], truth, seed)
        s["optics"] = o = [_optics(c, **t) for t in _midband_start(truth, seed)]
        s["ws"] = torch.empty(api.tune_workspace_size(o, 1), dtype=torch.uint8, device=DEV)
    elif kind == "restore":
        shapes = _restore_shapes(c)
        truth = _prior(c["n"], seed + 1)
        tiles = [_thin_stacks(z, y, x, 0.5 * max(y, x) / 128.0, truth[i:i + 1], seed + 10 * i)[0]
                 for i, (z, y, x) in enumerate(shapes)]
        s["d"] = api.pack_stacks(tiles)
        s["optics"] = o = [_optics(dict(nz=z, ny=y, nx=x, edge=0.5 * max(y, x) / 128.0)) for z, y, x in shapes]
        s["eta"] = [_thin_eta(z) for z, _, _ in shapes]
        off = np.random.default_rng(seed + 2).normal(size=(c["n"], 3)) * (0.1, 0.01, 0.02)
        th = np.concatenate([truth[:, :3] + off, truth[:, 3:]], 1)
        s["theta0"] = np.clip(th, (-2.5, 1.0, 0.0, -1.0), (2.5, 1.3, math.radians(32.0), 1.0))[:, None]
        s["ws"] = torch.empty(api.tune_workspace_size(o, 1), dtype=torch.uint8, device=DEV)
        s["f"] = torch.empty(sum(2 * y * x for _, y, x in shapes), device=DEV)
    elif kind == "cnn":
        s["params"], s["x"], s["t"] = _cnn_input(c, seed)
        s["ws"] = api.cnn_workspace(c["n"], (c["nz"], c["ny"], c["nx"]), DEV)
    else:
        x, w, gz = _conv_input(c, seed)
        s["x"], s["w"], s["gz"] = x.view(torch.int16), w.view(torch.int16), gz.view(torch.int16)
    return s


def _midband_start(truth, seed):
    """Parameters some way off the truth, as in the middle of a tune."""
    off = np.random.default_rng(seed + 3).normal(size=(len(truth), 3)) * (0.3, 0.02, 0.05)
    return [dict(defocus=float(t[0] + e[0]), na_det=float(np.clip(t[1] + e[1], 0.95, 1.28)),
                 tilt_zenith=float(np.clip(t[2] + e[2], 0.02, 0.55)), tilt_azimuth=0.05)
            for t, e in zip(truth, off)]


def run(s):
    api, c = s["api"], s["case"]
    kind = c["kind"]
    if kind == "step":
        if c["layout"] == "band":
            tf = api.transfer_function_band(s["optics"], out=s["tf"], ws=s["ws"])
            return {"f": api.linear_band(api.OP_RECONSTRUCT, s["optics"], tf, s["x"], s["eta"], ws=s["ws"]),
                    "tf": tf}
        tf = api.transfer_function(s["optics"], out=s["tf"], ws=s["ws"])
        return {"f": api.reconstruct(s["optics"], tf, s["x"], s["eta"], ws=s["ws"]), "tf": tf}
    if kind == "fwdadj":
        s["x"].grad = None
        d = api.linear_forward_fn(s["x"], s["optics"], s["tf"], s["b"])
        d.backward(s["g"])
        return {"d": d.detach(), "grad": s["x"].grad}
    if kind == "grad":
        s["x"].grad = s["theta"].grad = None
        f = api.reconstruct_fn(s["x"], s["theta"], s["optics"], s["eta"])
        f.backward(s["g"])
        # FP64 only in its container: the device computes in FP32
        return {"f": f.detach(), "grad_d": s["x"].grad, "grad_theta": s["theta"].grad.float()}
    if kind == "midband":
        loss, grad = api.midband_loss_grad(s["optics"], s["d"], _thin_eta(c["nz"]), NU_C, ws=s["ws"])
        return {"loss": loss.astype(np.float32), "grad": grad.astype(np.float32)}
    if kind == "restore":
        _, loss, theta, _, _ = api.restore_tiles(
            s["optics"], s["d"], s["eta"], iters=c["iters"], lr=(0.02, 0.005, 0.005, 0.001),
            lo=(-2.5, 1.0, 0.0, -1.0), hi=(2.5, 1.3, math.radians(32.0), 1.0), mask=0b0101,
            theta0=s["theta0"], nu_c=NU_C, use_graph=2, branches=8, f_out=s["f"], ws=s["ws"])
        return {"f": s["f"], "loss": loss.astype(np.float32), "theta": theta.astype(np.float32)}
    if kind == "cnn":
        y, loss, grad = api.cnn_gradient(s["params"], s["x"], s["t"], ws=s["ws"])
        return {"y": y, "loss": loss, "grad": grad}
    return {"z": api.conv3d_forward(s["x"], s["w"], c["cout"]),
            "gx": api.conv3d_input_grad(s["gz"], s["w"], tuple(s["x"].shape)),
            "gw": api.conv3d_weight_grad(s["x"], s["gz"])}


# ---------------------------------------------------------------- what a pass cannot do without

def _fft_flops(m):
    """Real transform of m values."""
    return 2.5 * m * math.log2(max(m, 2))


def _conv_flops(n, sizes, ci, co):
    return 2.0 * n * math.prod(sizes) * 27 * ci * co


def work(case):
    c = dict(case)
    kind = c["kind"]
    if kind in ("step", "fwdadj", "grad"):
        C, P = CHANNELS[c["model"]]
        V = c["n"] * c["nz"] * c["ny"] * c["nx"]
        H = c["n"] * c["nz"] * c["ny"] * (c["nx"] // 2 + 1)
        entries = 2 if c["model"] == "pol5" and c.get("layout") == "band" else C * P
        lin = (C + P) * _fft_flops(V) + H * (8 * C * P + 8 * C * P * P)
        syn = entries * _fft_flops(V)
        if kind == "step":
            # the band: the share of the frequencies within the pupils' support
            lam, px = (0.52 if c["model"] == "fluor" else 0.532), 0.1
            r = (2 * c["na_det"] if c["model"] == "fluor" else c["na_det"] + c["na_ill"]) / lam
            band = min(1.0, 2 * r * px) ** 2 if c["layout"] == "band" else 1.0
            return {"bytes": 4.0 * V * (C + P) + 8.0 * H * entries * band, "flops": lin + syn}
        if kind == "fwdadj":
            return {"bytes": 2 * 4.0 * V * (C + P) + 8.0 * H * C * P, "flops": 2 * lin}
        return {"bytes": 4.0 * V * (2 * C + 2 * P), "flops": 3 * lin + 3 * syn}
    if kind in ("midband", "restore"):
        shapes = [(c["nz"], c["ny"], c["nx"])] * c["n"] if kind == "midband" else _restore_shapes(c)
        iters = 1 if kind == "midband" else c["iters"] + 1
        V = sum(math.prod(s) for s in shapes)
        # two fields in, two real planes forward, the same back: four complex pairs of plane transforms
        flops = sum(iters * 6 * z * 5.0 * y * x * math.log2(y * x) for z, y, x in shapes)
        return {"bytes": 4.0 * V + (0 if kind == "midband" else sum(8.0 * y * x for _, y, x in shapes)),
                "flops": flops}
    if kind == "cnn":
        D, total, act = (c["nz"], c["ny"], c["nx"]), 0.0, 4.0 * c["n"] * c["nz"] * c["ny"] * c["nx"]
        for i, (ci, co) in enumerate(zip(CNN_CHANNELS[:-1], CNN_CHANNELS[1:])):
            D = tuple((v - 1) // 2 + 1 for v in D)
            total += (3 if i else 2) * _conv_flops(c["n"], D, ci, co)
        n = sum(co * (27 * ci + 1) for ci, co in zip(CNN_CHANNELS[:-1], CNN_CHANNELS[1:]))
        return {"bytes": act + 8.0 * n, "flops": total}
    out = _conv_sizes(c)
    xin, zout, w = c["n"] * c["nz"] * c["ny"] * c["nx"] * c["cin"], c["n"] * math.prod(out) * c["cout"], 27 * c["cin"] * c["cout"]
    return {"bytes": 2.0 * (xin + zout + w) + 4.0 * (xin + zout + w), "flops": 3 * _conv_flops(c["n"], out, c["cin"], c["cout"])}


# ---------------------------------------------------------------- the outputs in plain FP64

def _fftfreq(n, d):
    return torch.from_numpy(np.fft.fftfreq(n, d)).to(DEV)


def _disc(r2, radius, hw):
    """Pupil edge: hard disc on squared distances, or the C1 smoothstep of half-width hw."""
    if hw == 0.0:
        return (r2 <= radius * radius).to(torch.float64)
    r = torch.where(r2 > 0, r2, torch.ones_like(r2)).sqrt()
    r = torch.where(r2 > 0, r, torch.zeros_like(r))
    t = (((radius - r) / hw + 1) * 0.5).clamp(0, 1)
    return t * t * (3 - 2 * t)


def _pupils(c, theta, wavelength=0.532):
    """S, P (n, Y, X), kz, km and the frequencies for theta (n, 4) float64."""
    ny, nx = c["ny"], c["nx"]
    fy, fx = _fftfreq(ny, 0.1)[:, None], _fftfreq(nx, 0.1)[None, :]
    km = 1.33 / wavelength
    hw = c["edge"] * min(1.0 / (nx * 0.1), 1.0 / (ny * 0.1))
    r2 = fy * fy + fx * fx
    kz = (km * km - r2).clamp(min=0).sqrt()
    na, zen, az = (theta[:, j, None, None] for j in (1, 2, 3))
    P = _disc(r2.expand(len(theta), ny, nx), na / wavelength, hw)
    q = km * torch.sin(zen)
    dy, dx = fy - q * torch.sin(az), fx - q * torch.cos(az)
    S = _disc(dy * dy + dx * dx, c.get("na_ill", 0.5) / wavelength, hw)
    return S, P, kz, km, fy, fx, dy, dx


def _arms(c, theta, z):
    """Spectra of the direct and scattered arms (n, Z, Y, X) and the scale Y X / I_bg."""
    S, P, kz, km, *_ = _pupils(c, theta)
    g = torch.where(kz > 0, km / torch.where(kz > 0, kz, torch.ones_like(kz)), torch.zeros_like(kz))
    prop = torch.exp(2j * math.pi * kz * (z[None, :, None, None] - theta[:, 0, None, None, None]))
    ibg = (S * P * P).sum((1, 2))
    return (S * P)[:, None] * prop, (P * g)[:, None] * 1j * prop, c["ny"] * c["nx"] / ibg



def _planes(c):
    return _fftfreq(c["nz"], 1.0) * c["nz"] * c["dz"]


def _kappa():
    """Coupling of the five swing states and the states themselves."""
    e0 = np.array([1.0, 1.0j]) / math.sqrt(2.0)
    d = math.pi * SWING
    states = [e0]
    for a in (0.0, math.pi / 4, math.pi / 2, 3 * math.pi / 4):
        rot = np.array([[math.cos(a), math.sin(a)], [-math.sin(a), math.cos(a)]])
        states.append(rot.T @ np.diag([np.exp(-1j * d), np.exp(1j * d)]) @ rot @ e0)
    a = np.array([1.0, -1.0j]) / math.sqrt(2.0)
    B = [np.eye(2), np.diag([0.5, -0.5]), np.array([[0, 0.5], [0.5, 0]]), 1j * np.eye(2)]
    k = np.array([[np.conj(a.conj() @ e) * (a.conj() @ (b @ e)) for b in B] for e in states])
    return k, states, a


def _sh(code):
    e = np.eye(3)
    x, y, z = e
    o = np.outer
    Y = {0: e, 4: 0.5 * (o(x, y) + o(y, x)), 8: 0.5 * (o(x, x) - o(y, y))}[code // 2]
    return Y * (1j if code % 2 else 1.0)


def _pair(c, theta):
    """[H_phase, H_abs] half spectra (Z, Y, Xh) of one patch's 3D label-free model."""
    a, b, s = _arms(c, theta, _planes(c))
    r = torch.fft.ifft2(b[0]) * torch.fft.ifft2(a[0]).conj() * s[0]
    return [torch.fft.rfftn(2 * r.real), torch.fft.rfftn(-2 * r.imag)]


def _vector_bank(c, theta):
    S, P, kz, km, fy, fx, *_ = _pupils(c, theta)
    S, P = S[0], P[0]
    ibg = (S * P * P).sum()
    w = 1.0 / (km * (km + kz))
    one, fyb, fxb = torch.ones_like(kz), fy.expand_as(kz), fx.expand_as(kz)
    Q = [[1 - fx * fx * w, -fx * fy * w], [-fx * fy * w, 1 - fy * fy * w], [-fxb / km, -fyb / km]]
    k = [fxb / km, fyb / km, kz / km]
    g = torch.where(kz > 0, km / torch.where(kz > 0, kz, one), torch.zeros_like(kz)) * 1j
    U = [[P * g * sum(Q[j][i] * ((j == n) * one - k[j] * k[n]) for j in range(3)) for n in range(3)] for i in range(2)]
    if c["model"] == "vector5":
        _, states, a = _kappa()
        chans = [(e, np.outer(a, a.conj())) for e in states]
    else:
        J = np.array([1.0, 1.0j]) / math.sqrt(2.0)
        sig = [np.eye(2), np.diag([1.0, -1.0]), np.array([[0, 1], [1, 0]]), np.array([[0, -1j], [1j, 0]])]
        chans = [(J, m) for m in sig]
    T = [_sh(code) for code in VEC_PROPS]
    Z, Y, X = c["nz"], c["ny"], c["nx"]
    out = [[torch.empty((Z, Y, X), dtype=torch.float64, device=DEV) for _ in T] for _ in chans]
    zs = _planes(c)
    step = max(1, int(2 ** 22 // (Y * X)))
    for z0 in range(0, Z, step):
        prop = torch.exp(2j * math.pi * kz * (zs[z0:z0 + step, None, None] - theta[0, 0]))
        u = [[torch.fft.ifft2(U[i][n] * prop) for n in range(3)] for i in range(2)]
        last = None
        for ci, (J, M) in enumerate(chans):
            if last is None or not np.array_equal(J, last):
                wk = [torch.fft.ifft2(S * P * (Q[m][0] * J[0] + Q[m][1] * J[1]).conj() * prop).conj()
                      for m in range(3)]
                last = J
            alpha = J.conj() @ M
            beta = [alpha[0] * u[0][n] + alpha[1] * u[1][n] for n in range(3)]
            for p, t in enumerate(T):
                r = sum(t[n, m] * beta[n] * wk[m] for n in range(3) for m in range(3) if t[n, m] != 0)
                out[ci][p][z0:z0 + step] = 2 * (r * (Y * X / ibg)).real
    for row in out:
        for p in range(len(row)):
            row[p] = torch.fft.rfftn(row[p])
    return out


def _sector(dy, dx):
    """Azimuthal eighth of (dy, dx) from +x towards +y, the origin in sector 0."""
    k = torch.full_like(dy, 6, dtype=torch.int64)
    q0, q1, q2 = (dy >= 0) & (dx > 0), (dx <= 0) & (dy > 0), (dy <= 0) & (dx < 0)
    q3 = ~(q0 | q1 | q2)
    for q, cond, i, j in ((q0, dy < dx, 0, 1), (q1, dy > -dx, 2, 3), (q2, dy > dx, 4, 5), (q3, dx < -dy, 6, 7)):
        k = torch.where(q, torch.where(cond, i, j), k)
    return torch.where((dy == 0) & (dx == 0), torch.zeros_like(k), k)


def _bank(c, theta):
    """(C lists of P) half spectra (Z, Y, Xh); the polarisation model's pair with its coupling."""
    m = c["model"]
    if m == "labelfree":
        return [_pair(c, theta)]
    if m == "pol5":
        return _pair(c, theta)
    if m.startswith("vector"):
        return _vector_bank(c, theta)
    zs = _planes(c)
    if m == "fluor":
        _, P, kz, *_ = _pupils(c, theta, 0.52)
        h = torch.fft.ifft2(P * torch.exp(2j * math.pi * kz * (zs[:, None, None] - theta[0, 0])))
        psf = h.abs() ** 2
        return [[torch.fft.rfftn(psf / psf.sum())]]
    S, P, kz, km, _, _, dy, dx = _pupils(c, theta)
    S, P = S[0], P[0]
    sec = _sector((dy + 0 * dx)[0], (dx + 0 * dy)[0])
    prop = torch.exp(2j * math.pi * kz * (zs[:, None, None] - theta[0, 0]))
    g = torch.where(kz > 0, km / torch.where(kz > 0, kz, torch.ones_like(kz)), torch.zeros_like(kz)) * 1j
    b = torch.fft.ifft2(P * g * prop)
    out = []
    for ch in range(9):
        Sc = S if ch == 8 else S * (sec == ch)
        r = b * torch.fft.ifft2(Sc * P * prop).conj() * (c["ny"] * c["nx"] / (Sc * P * P).sum())
        out.append([torch.fft.rfftn(2 * r.real)])
    return out


def _entry(c, bank, z):
    """The bank's entries H[c][p] on the planes z (a slice)."""
    if c["model"] == "pol5":
        k, u, v = _kappa()[0], bank[0][z], bank[1][z]
        return [[k[i, p].real * u + k[i, p].imag * v for p in range(4)] for i in range(5)]
    return [[h[z] for h in row] for row in bank]


def _tikhonov(H, D, eta):
    """F = (H^H H + eta)^-1 H^H D by Cholesky, entry by entry."""
    C, P = len(H), len(H[0])
    rhs = [sum(H[i][p].conj() * D[i] for i in range(C)) for p in range(P)]
    M = [[sum(H[i][p].conj() * H[i][q] for i in range(C)) for q in range(p + 1)] for p in range(P)]
    L, inv = [[None] * P for _ in range(P)], [None] * P
    for j in range(P):
        d = M[j][j].real + eta - sum((L[j][k].real ** 2 + L[j][k].imag ** 2 for k in range(j)), 0.0)
        inv[j] = d.rsqrt()
        for i in range(j + 1, P):
            L[i][j] = (M[i][j] - sum((L[i][k] * L[j][k].conj() for k in range(j)), 0.0)) * inv[j]
    y = []
    for j in range(P):
        y.append((rhs[j] - sum((L[j][k] * y[k] for k in range(j)), 0.0)) * inv[j])
    x = [None] * P
    for j in reversed(range(P)):
        x[j] = (y[j] - sum((L[k][j].conj() * x[k] for k in range(j + 1, P)), 0.0)) * inv[j]
    return x


def _theta(o):
    return torch.tensor([[o.defocus, o.na_det, o.tilt_zenith, o.tilt_azimuth]], dtype=torch.float64, device=DEV)


def _exact_linear(c, seed):
    x = _linear_input(c, seed)
    vol = (c["nz"], c["ny"], c["nx"])
    C, P = CHANNELS[c["model"]]
    up = _volume((c["n"], C) + vol, seed + 1, 0.01) if c["kind"] == "fwdadj" else None
    first, second, banks = [], [], []
    chunk = max(1, int(2 ** 22 // (vol[1] * vol[2])))
    for i, o in enumerate(_patches(c)):
        bank = _bank(c, _theta(o))
        ins = [torch.fft.rfftn(v.double()) for v in x[i]]
        gs = [torch.fft.rfftn(v.double()) for v in up[i]] if up is not None else None
        outs = [torch.empty_like(ins[0]) for _ in range(P if gs is None else C)]
        adj = [torch.empty_like(ins[0]) for _ in range(P)] if gs is not None else None
        for z0 in range(0, vol[0], chunk):
            z = slice(z0, z0 + chunk)
            H = _entry(c, bank, z)
            if gs is None:
                for p, v in enumerate(_tikhonov(H, [d[z] for d in ins], _eta(c))):
                    outs[p][z] = v
            else:
                for k in range(C):
                    outs[k][z] = sum(H[k][p] * ins[p][z] for p in range(P))
                for p in range(P):
                    adj[p][z] = sum(H[k][p].conj() * gs[k][z] for k in range(C))
        b = 0.01 if gs is not None else 0.0
        first.append(torch.stack([torch.fft.irfftn(v, s=vol) + b for v in outs]))
        if adj is not None:
            second.append(torch.stack([torch.fft.irfftn(v, s=vol) for v in adj]))
        elif c["layout"] == "full":
            banks.append(torch.stack([torch.stack([h for h in row]) for row in _entry(c, bank, slice(None))]))
    if c["kind"] == "fwdadj":
        return {"d": torch.stack(first), "grad": torch.stack(second)}
    # in the band layout the bank's place has a layout of the library's own choice
    return {"f": torch.stack(first), "tf": torch.stack(banks) if banks else None}


def _exact_grad(c, seed):
    x = _linear_input(c, seed).double()
    vol = (c["nz"], c["ny"], c["nx"])
    up = _volume((c["n"], 2) + vol, seed + 1, 0.01) * 1e-4
    f, gd, gt = [], [], []
    for i, o in enumerate(_patches(c)):
        th, d = _theta(o).requires_grad_(True), x[i].clone().requires_grad_(True)
        H = [_pair(c, th)]
        F = _tikhonov(H, [torch.fft.rfftn(d[0])], _eta(c))
        fi = torch.stack([torch.fft.irfftn(v, s=vol) for v in F])
        fi.backward(up[i].double())
        f.append(fi.detach())
        gd.append(d.grad)
        gt.append(th.grad[0].cpu())
    return {"f": torch.stack(f), "grad_d": torch.stack(gd), "grad_theta": torch.stack(gt)}


def _exact_midband(c, seed):
    truth = _prior(c["n"], seed + 1)
    d = _thin_stacks(c["nz"], c["ny"], c["nx"], c["edge"], truth, seed)
    start = np.array([[t["defocus"], t["na_det"], t["tilt_zenith"], t["tilt_azimuth"]]
                      for t in _midband_start(truth, seed)])
    fy, fx = _fftfreq(c["ny"], 0.1)[:, None], _fftfreq(c["nx"], 0.1)[None, :]
    r = (fy * fy + fx * fx).sqrt()
    band = (r >= NU_C / 8) & (r <= NU_C / 4)
    z = 0.2 * (torch.arange(c["nz"], device=DEV, dtype=torch.float64) - (c["nz"] - 1) / 2)
    losses, grads = [], []
    step = max(1, int(2 ** 22 // (c["nz"] * c["ny"] * c["nx"])))
    for i in range(0, c["n"], step):
        th = torch.from_numpy(start[i:i + step]).to(DEV).requires_grad_(True)
        a, b, s = _arms(c, th, z)
        cz = torch.fft.ifft2(b) * torch.fft.ifft2(a).conj() * s[:, None, None, None]
        hp, ha = torch.fft.fft2(2 * cz.real)[..., band], torch.fft.fft2(-2 * cz.imag)[..., band]
        D = torch.fft.fft2(d[i:i + step].double())[..., band]
        H = [[hp[:, k], ha[:, k]] for k in range(c["nz"])]
        F = _tikhonov(H, [D[:, k] for k in range(c["nz"])], _thin_eta(c["nz"]))[0]
        loss = -(F.real ** 2 + F.imag ** 2).mean(1)
        loss.sum().backward()
        losses.append(loss.detach().cpu())
        grads.append(th.grad.cpu())
    return {"loss": torch.cat(losses).numpy(), "grad": torch.cat(grads).numpy()}


def _conv3(x, w):
    """Channels-last convolution (stride 2, padding 1) in FP64: one product per tap."""
    n, D, H, W, ci = x.shape
    co = w.shape[0]
    xp = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1, 1, 1))
    Do, Ho, Wo = (D - 1) // 2 + 1, (H - 1) // 2 + 1, (W - 1) // 2 + 1
    w = w.reshape(co, 27, ci)
    z = 0.0
    for t in range(27):
        kd, kh, kw = t // 9, t // 3 % 3, t % 3
        patch = xp[:, kd:kd + 2 * Do - 1:2, kh:kh + 2 * Ho - 1:2, kw:kw + 2 * Wo - 1:2]
        z = z + patch.reshape(-1, ci) @ w[:, t].t()
    return z.reshape(n, Do, Ho, Wo, co)


def _exact_cnn(c, seed):
    """The network in FP64 throughout (no rounding of activations or weights)."""
    params, x, t = _cnn_input(c, seed)
    p = params.double().requires_grad_(True)
    x = x.double()
    a = (x / (x * x).mean((1, 2, 3), keepdim=True).sqrt())[..., None]
    off = 0
    for ci, co in zip(CNN_CHANNELS[:-1], CNN_CHANNELS[1:]):
        w, b = p[off:off + co * 27 * ci].reshape(co, 27 * ci), p[off + co * 27 * ci:off + co * (27 * ci + 1)]
        off += co * (27 * ci + 1)
        a = torch.nn.functional.gelu(_conv3(a, w) + b)
    y = a.mean((1, 2, 3)) @ p[off:off + 768].reshape(3, 256).t() + p[off + 768:]
    loss = ((y - t.double()) ** 2).mean()
    loss.backward()
    return {"y": y.detach(), "loss": loss.detach().reshape(1), "grad": p.grad}


def exact(case, seed):
    c = dict(case)
    kind = c["kind"]
    if kind in ("step", "fwdadj"):
        return _exact_linear(c, seed)
    if kind == "grad":
        return _exact_grad(c, seed)
    if kind == "midband":
        return _exact_midband(c, seed)
    if kind == "cnn":
        return _exact_cnn(c, seed)
    if kind == "conv":
        x, w, gz = (v.double() for v in _conv_input(c, seed))
        x.requires_grad_(True)
        w.requires_grad_(True)
        z = _conv3(x, w)
        z.backward(gz)
        return {"z": z.detach(), "gx": x.grad, "gw": w.grad}
    return None   # a whole tune: 20 iterations of every tile's loss and gradient in FP64 take minutes
