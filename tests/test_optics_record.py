"""The record path of the optics marshalling writes the bytes of the field-by-field
path, and hands over to it whatever it cannot take (CPU)."""

import dataclasses

import numpy as np
import pytest

from paper_2412_09775_amd import api

BASE = api.Optics(model=5, nz=9, ny=64, nx=32, dz=0.2, dy=0.1, dx=0.1, wavelength=0.53, na_ill=0.5, na_det=1.1,
                  n_medium=1.33, defocus=-0.3, tilt_zenith=0.1, tilt_azimuth=0.2, edge_width=0.5, swing=0.03,
                  zernike=(0.1, -0.2, 0.3), det_tilt=0.01, det_azimuth=0.02, vec_channels=1, vec_props=(0, 17, 3),
                  ill_jones=(0.6 + 0.1j, -0.5))

FORMS = {
    "plain": {}, "no_aberration": dict(zernike=()), "none_aberration": dict(zernike=None),
    "seven_terms": dict(zernike=(1, 2, 3, 4, 5, 6, 7)), "array_terms": dict(zernike=np.array([0.25, 0.5])),
    "numpy_numbers": dict(nz=np.int64(7), dz=np.float32(0.2), model=np.int32(3)), "float_sizes": dict(nz=8.0),
    "text_number": dict(dz="0.5"), "eight_props": dict(vec_props=tuple(range(8))), "list_props": dict(vec_props=[1, 2]),
    "bool_model": dict(model=True), "nan": dict(defocus=float("nan")), "infinite": dict(edge_width=float("inf")),
    "real_jones": dict(ill_jones=(1, 0)), "wide_size": dict(nz=2 ** 40),
}


@pytest.mark.parametrize("name", FORMS)
def test_bytes(name):
    o = dataclasses.replace(BASE, **FORMS[name])
    want = (api.WoOptics * 1)()
    api._fill_fields(want, 0, o)
    assert bytes(api.optics_array(o)) == bytes(want)
    as_dict = {f.name: getattr(o, f.name) for f in dataclasses.fields(o)}
    assert bytes(api.optics_array([as_dict])) == bytes(want)


@pytest.mark.parametrize("bad", [dict(zernike=(0,) * 8), dict(vec_props=(0,) * 9), dict(nz="x"), dict(ill_jones=(1,)),
                                 dict(dz=None)])
def test_refused_as_before(bad):
    o = dataclasses.replace(BASE, **bad)
    with pytest.raises((ValueError, TypeError)) as want:
        api._fill_fields((api.WoOptics * 1)(), 0, o)
    with pytest.raises(type(want.value)):
        api.optics_array(o)
