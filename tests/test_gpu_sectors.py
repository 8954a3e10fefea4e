"""The nine-aperture bank through the shared scattered arm vs the FP64 oracle.

Shapes around the row kernel's choices: several rows a workgroup, one, lines in
two batches (1024 points), row lengths without compiled stages, rows too long for
one workgroup (the pairwise pass), the support filling the grid; tilt, defocus,
aberrations and two patches.  Relative L2 <= 1e-5 per channel, as for every bank."""

import numpy as np
import pytest

from oracle import optics as op
from oracle import tf as tfm

pytestmark = pytest.mark.gpu

CASES = {
    "rows_of_64": dict(shape=(5, 60, 64)),
    "rows_of_192": dict(shape=(4, 48, 240), zernike=(0.05, 0.0, -0.04)),
    "two_batches": dict(shape=(2, 40, 1200), na_det=1.2),
    "runtime_length": dict(shape=(6, 36, 50), dx=0.12),
    "long_rows": dict(shape=(2, 24, 2400), na_det=1.2, na_ill=0.9),
    "fills_grid": dict(shape=(4, 32, 40), dx=0.155),
}


@pytest.mark.parametrize("name", CASES)
def test_bank(gpu_lib, name):
    c = dict(CASES[name])
    nz, ny, nx = c.pop("shape")
    base = dict(model=op.SECTORS9_3D, nz=nz, ny=ny, nx=nx, dz=0.2, dy=c.get("dx", 0.1), dx=0.1, wavelength=0.532,
                na_ill=0.6, na_det=1.0, n_medium=1.33, tilt_zenith=0.05, tilt_azimuth=0.4, defocus=0.1)
    base.update(c)
    from paper_2412_09775_amd import api
    os_ = [op.Optics(**base), op.Optics(**dict(base, defocus=-0.2, na_det=base["na_det"] * 0.97))]
    print(f"[case] sectors {name} {(nz, ny, nx)}", flush=True)
    got = gpu_lib.transfer_function([api.Optics(**{k: getattr(o, k) for k in base}) for o in os_],
                                    device="cuda:0").cpu().numpy()
    for i, o in enumerate(os_):
        ref = tfm.transfer_function(o)[..., : nx // 2 + 1]
        err = [np.linalg.norm(got[i, ch] - ref[ch]) / np.linalg.norm(ref[ch]) for ch in range(9)]
        print(f"  patch {i}: worst channel rel L2 {max(err):.2e}", flush=True)
        assert max(err) <= 1e-5
