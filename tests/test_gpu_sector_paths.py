"""Which nine-aperture calls go through the shared scattered arm, and their banks.

The shared arm serves many rows, of compiled lengths or of others that fill the chip,
and rows beyond 1024 points; small banks and the other rows on the runtime plan, which
it slowed down, take the pairwise rows.  Shapes on both sides of the rule, the shared
kernel's choices among them (several rows a workgroup, one, lines in two batches, the
runtime plan): the kernels that ran, and the bank against the FP64 oracle at relative
L2 <= 1e-5 per channel, as for every bank."""

import numpy as np
import pytest

from oracle import optics as op
from oracle import tf as tfm

pytestmark = pytest.mark.gpu

# shape, patches, shared arm expected, row length, options
CASES = [((32, 60, 64), 1, False, 64, {}), ((36, 60, 64), 1, True, 64, {}), ((18, 60, 64), 2, True, 64, {}),
         ((4, 36, 40), 1, False, 40, dict(dx=0.155)), ((45, 48, 240), 1, True, 160, dict(zernike=(0.05, 0.0, -0.04))),
         ((64, 48, 100), 1, True, 100, dict(na_det=1.15)), ((64, 48, 120), 1, False, 120, dict(na_det=1.1, dx=0.12)), ((54, 40, 1200), 1, True, 1024, dict(na_det=1.2)),
         ((40, 54, 400), 1, True, 240, dict(na_det=0.7, edge_width=0.5)), ((3, 32, 1500), 1, True, 1500, dict(na_det=1.2))]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c[0])))
def test_path_and_bank(gpu_lib, case):
    from paper_2412_09775_amd import api
    (nz, ny, nx), n, shared, lx, opts = case
    opts = dict(opts)
    base = dict(model=op.SECTORS9_3D, nz=nz, ny=ny, nx=nx, dz=0.2, dy=opts.get("dx", 0.1), dx=0.1, wavelength=0.532,
                na_ill=0.6, na_det=1.0, n_medium=1.33, tilt_zenith=0.05, tilt_azimuth=0.4, defocus=0.1)
    base.update(opts)
    os_ = [op.Optics(**dict(base, defocus=0.1 - 0.3 * i)) for i in range(n)]
    optics = [api.Optics(**{k: getattr(o, k) for k in base}) for o in os_]
    print(f"[case] sector paths {(nz, ny, nx)} x {n}", flush=True)
    assert api.lateral_support(optics)["tf_lengths"][1] == lx
    gpu_lib.timing_enable(True)
    gpu_lib.timing_report()
    got = gpu_lib.transfer_function(optics, device="cuda:0").cpu().numpy()
    ran = gpu_lib.timing_report()
    gpu_lib.timing_enable(False)
    assert ("k_tf_rows_sectors" in ran) == shared and ("k_tf_rows_lf" in ran) != shared
    for i, o in enumerate(os_):
        ref = tfm.transfer_function(o)[..., : nx // 2 + 1]
        err = [np.linalg.norm(got[i, ch] - ref[ch]) / np.linalg.norm(ref[ch]) for ch in range(9)]
        print(f"  patch {i}: worst channel rel L2 {max(err):.2e}", flush=True)
        assert max(err) <= 1e-5
