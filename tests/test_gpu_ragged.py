"""Transforms of ragged lengths through the linear calls.

The forward model and the reconstruction of random volumes against numpy FP64
transforms with the same bank (the library's own, so only the transforms and the
per-frequency step are compared).  Row and column lengths with compiled stages over
every radix of their plans (2 to 12), one to four passes, odd and even first radices,
several rows a workgroup and one; a few shapes (Z below 16, rows of 30, 1152, 2048 and
4096 points) take the runtime plans, of radices 2, 3, 4, 5 and 8.  Relative L2 <= 1e-5
(FP32 transforms) and 1e-4 (solve), the bounds of the parity suite."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# (nz, ny, nx): X rows, Y and Z columns
SHAPES = [(1, 40, 50), (2, 54, 72), (3, 60, 90), (5, 50, 100), (9, 48, 108), (10, 36, 150), (12, 90, 162), (15, 40, 200),
          (18, 72, 216), (25, 54, 250), (27, 40, 270), (4, 270, 54), (6, 36, 288), (8, 450, 36), (45, 30, 40),
          (75, 40, 36), (81, 36, 40), (125, 32, 36), (20, 30, 300), (3, 40, 360), (2, 500, 40), (3, 32, 400),
          (2, 36, 432), (3, 40, 450), (2, 30, 486), (2, 36, 540), (3, 40, 576), (2, 648, 32), (2, 40, 600), (2, 36, 640),
          (2, 40, 720), (2, 36, 750), (3, 32, 768), (2, 810, 30), (2, 30, 864), (2, 36, 900), (2, 40, 972),
          (2, 32, 1000), (2, 1152, 32), (1, 40, 2048), (1, 2048, 40), (1, 32, 4096), (100, 30, 32), (90, 32, 30)]


@pytest.mark.parametrize("shape", SHAPES)
def test_linear_calls(gpu_lib, shape):
    import torch
    from paper_2412_09775_amd import api
    nz, ny, nx = shape
    # a wide pupil on a coarse grid: the band takes most of it
    o = api.Optics(model=api.MODEL_LABELFREE_3D, nz=nz, ny=ny, nx=nx, dz=0.2, dy=0.13, dx=0.13, wavelength=0.532,
                   na_ill=0.7, na_det=1.1, n_medium=1.33, edge_width=0.3)
    print(f"[case] ragged {shape}", flush=True)
    rng = np.random.default_rng(nz * 7919 + ny * 31 + nx)
    f = rng.standard_normal((2, nz, ny, nx)).astype(np.float32)
    d = rng.standard_normal((1, nz, ny, nx)).astype(np.float32)
    tf = gpu_lib.transfer_function([o], device="cuda:0")
    bank = tf.cpu().numpy()[0, 0].astype(np.complex128)
    eta = 1e-2 * float(np.max(np.sum(np.abs(bank) ** 2, axis=0)))
    got_d = gpu_lib.forward([o], tf, torch.from_numpy(f[None]).cuda()).cpu().numpy()[0, 0]
    got_f = gpu_lib.reconstruct([o], tf, torch.from_numpy(d[None]).cuda(), eta).cpu().numpy()[0]
    ref_d = np.fft.irfftn(np.sum(bank * np.fft.rfftn(f.astype(np.float64), axes=(1, 2, 3)), axis=0),
                          s=(nz, ny, nx), axes=(0, 1, 2))
    D = np.fft.rfftn(d[0].astype(np.float64), axes=(0, 1, 2))
    F = np.conj(bank) * D / (np.sum(np.abs(bank) ** 2, axis=0) + eta)
    ref_f = np.fft.irfftn(F, s=(nz, ny, nx), axes=(1, 2, 3))
    ed = np.linalg.norm(got_d - ref_d) / np.linalg.norm(ref_d)
    ef = np.linalg.norm(got_f - ref_f) / np.linalg.norm(ref_f)
    print(f"  forward {ed:.2e} reconstruct {ef:.2e}", flush=True)
    assert ed <= 1e-5 and ef <= 1e-4
