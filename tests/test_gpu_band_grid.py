"""The auto-tune's loss and gradient on the loss band's own grid vs the FP64 oracle.

The iterations sample the field of view on the shortest transform lengths at which
the band's transfer function is exact; the oracle works on the full grid.  Shapes
around the choice of the length (shortened on both axes, on one, ragged, none),
bands from a few frequencies to the whole grid, steep tilt at high aperture (the
widest spectra), and patches of one call with different bands.  Tolerances as for
the loss and gradient everywhere (FP32 transforms of condition up to sigma^2 / eta
= 100): 1e-4 and 1e-3."""

import numpy as np
import pytest

import synth
from oracle import autotune as at
from oracle import linear
from oracle import optics as op
from oracle import tf as tfm

pytestmark = pytest.mark.gpu

CASES = {
    "both_axes": dict(shape=(8, 128, 128), nu=(0.0,)),
    "ragged": dict(shape=(5, 100, 150), nu=(0.0,)),
    "one_axis": dict(shape=(6, 54, 160), nu=(0.0,)),
    "odd_planes": dict(shape=(3, 160, 96), nu=(0.0, 2.0)),
    "narrow_band": dict(shape=(4, 128, 96), nu=(0.7,)),
    "wide_band": dict(shape=(4, 128, 128), nu=(9.0, 1.5)),
    "whole_grid": dict(shape=(4, 64, 80), nu=(19.0,)),
    "steep": dict(shape=(4, 192, 128), nu=(0.0,), tilt=0.55, na=1.28),
}


@pytest.mark.parametrize("name", CASES)
def test_loss_and_gradient(gpu_lib, name):
    import torch
    c = CASES[name]
    nz, ny, nx = c["shape"]
    base = op.Optics(model=op.LABELFREE_THIN, nz=nz, ny=ny, nx=nx, dz=0.4, dy=0.1, dx=0.1, wavelength=0.532,
                     na_ill=0.5, na_det=c.get("na", 1.15), n_medium=1.33, tilt_zenith=c.get("tilt", 0.2),
                     tilt_azimuth=0.3, edge_width=0.5 * max(ny, nx) / 128.0, defocus=0.15)
    truth = base.replace(defocus=-0.4, tilt_zenith=0.1)
    bank = tfm.labelfree_thin(truth)
    eta = 1e-2 * linear.max_singular_value_sq(bank)
    opts, stacks, nus = [], [], []
    for i, nu in enumerate(c["nu"]):
        f = synth.thin_cells((ny, nx), 0.1, 8, seed=900 + i)
        stacks.append((linear.forward(bank, f) + synth.gaussian_noise((nz, ny, nx), 2e-3, 910 + i)).astype(np.float32))
        opts.append(base)
        nus.append(nu if nu > 0 else at.nominal_cutoff(base))
    print(f"[case] band grid {name} {c['shape']} nu_c {nus}", flush=True)
    loss, grad = gpu_lib.midband_loss_grad(opts, torch.from_numpy(np.stack(stacks)).cuda(), eta, np.array(nus))
    for i, o in enumerate(opts):
        L, g = at.loss_and_gradient(o, stacks[i].astype(np.float64), eta, nus[i])
        el, eg = abs(loss[i] - L) / abs(L), np.max(np.abs(grad[i] - g)) / np.max(np.abs(g))
        print(f"  patch {i}: loss rel {el:.2e} grad rel {eg:.2e}", flush=True)
        assert el < 1e-4 and eg < 1e-3
