"""The batch sizes at which the launch settings change, asked of the library on the host, against the
sizes at which the settings were measured to change places on MI355X."""
import ctypes

import pytest

from paper_2604_19906_amd import tpo

DT = {"f64": (tpo.TPO_F64, 8), "f32": (tpo.TPO_F32, 4)}


def conv_elems(dtype, nv, nq, mb):
    return int(mb * 1e6 / ((10 * nq ** 3 + 3 * nv ** 3) * DT[dtype][1]))


@pytest.fixture(scope="module")
def convection_setting():
    fn = tpo.lib().tpo_internal_convection_setting
    fn.argtypes = [ctypes.c_int] * 3 + [ctypes.c_longlong]
    return lambda dtype, nv, nq, mb: fn(nv, nq, DT[dtype][0], conv_elems(dtype, nv, nq, mb))


# all loads first: 1.06 .. 1.09 of the time of the other form at 275 .. 340 MB for n = 11, 0.96 at 1.2 GB
@pytest.mark.parametrize("n,keeps,takes", [(11, 800, 1200), (12, 500, 1200), (13, 240, 600),
                                           (14, 240, 380), (15, 240, 275), (16, 240, 275)])
def test_convection_f64_loads_first(convection_setting, n, keeps, takes):
    assert convection_setting("f64", n, n, keeps) == 0
    assert convection_setting("f64", n, n, takes) == 1
