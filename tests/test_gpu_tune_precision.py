"""Rounding error of the mid-band loss and gradient on the band's own grid.

A grid of fewer points averages the rounding of fewer points and has to make up for
it: iterations on the tile's own grid, with the radices and twiddles of its length,
were off from FP64 by 2.7e-7 to 4.9e-7 of the gradients' norm on these batches of
patches (random optics some way off the truth); on the band's grid 4.3e-7 to 7.1e-7
with twiddles formed as powers and FP32 normal matrices, 2.4e-7 to 3.2e-7 without.
Bound: 4.5e-7; for the loss 2.5e-7, a few units of FP32."""

import math

import numpy as np
import pytest

import synth
from oracle import autotune as at
from oracle import linear
from oracle import optics as op
from oracle import tf as tfm

pytestmark = pytest.mark.gpu

NU_C = (1.15 + 0.5) / 0.532


@pytest.mark.parametrize("shape", [(10, 80, 120), (15, 144, 144), (15, 108, 192)])
def test_gradient_error(gpu_lib, shape):
    import torch
    nz, ny, nx = shape
    n = 24
    rng = np.random.default_rng(nz * ny + nx)
    base = op.Optics(model=op.LABELFREE_THIN, nz=nz, ny=ny, nx=nx, dz=0.2, dy=0.1, dx=0.1, wavelength=0.532,
                     na_ill=0.5, na_det=1.15, n_medium=1.33, edge_width=0.5 * max(ny, nx) / 128.0)
    opts, stacks = [], []
    for i in range(n):
        z, na, tilt = rng.uniform(-2, 2), rng.uniform(0.98, 1.27), rng.uniform(0, math.radians(30))
        d = linear.forward(tfm.labelfree_thin(base.replace(defocus=z, na_det=na, tilt_zenith=tilt)),
                           synth.thin_cells((ny, nx), 0.1, 12, seed=100 + i))
        stacks.append((d + synth.gaussian_noise((nz, ny, nx), 0.03, 300 + i)).astype(np.float32))
        off = rng.normal(size=3) * (0.3, 0.02, 0.05)
        opts.append(base.replace(defocus=z + off[0], na_det=float(np.clip(na + off[1], 0.95, 1.28)),
                                 tilt_zenith=float(np.clip(tilt + off[2], 0.02, 0.55)), tilt_azimuth=0.05))
    eta = 0.05 * nz
    print(f"[case] tune precision {shape}", flush=True)
    loss, grad = gpu_lib.midband_loss_grad(opts, torch.from_numpy(np.stack(stacks)).cuda(), eta, np.full(n, NU_C))
    ref = [at.loss_and_gradient(o, d.astype(np.float64), eta, NU_C) for o, d in zip(opts, stacks)]
    L, G = np.array([r[0] for r in ref]), np.array([r[1] for r in ref])
    el, eg = np.linalg.norm(loss - L) / np.linalg.norm(L), np.linalg.norm(grad - G) / np.linalg.norm(G)
    print(f"  loss {el:.2e} gradient {eg:.2e}", flush=True)
    assert eg < 4.5e-7 and el < 2.5e-7
