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


# (dtype, nv, nq), MB of fields on which the utilisation rule's setting leads, on which the table's does
@pytest.mark.parametrize("dtype,nv,nq,rule,row", [
    ("f64", 6, 8, (100, 275, 310), (600, 2500)), ("f64", 7, 8, (100, 275, 310), (380, 2500)),
    ("f64", 7, 9, (100, 275, 310), (380, 2500)), ("f64", 9, 11, (100, 275, 310), (340, 2500)),
    ("f64", 8, 12, (100, 240), (340, 2500)), ("f64", 12, 14, (1, 300, 2500), ()),
    ("f64", 8, 10, (), (1, 16, 200, 2500)), ("f64", 11, 12, (), (1, 16, 200, 2500)),
    ("f32", 2, 3, (100, 275, 310), (430, 2500)), ("f32", 3, 4, (100, 275, 310), (340, 2500)),
    ("f32", 6, 9, (13, 16, 23), (30, 60, 240)),
    ("f32", 8, 10, (13, 15, 18), (4, 11, 20, 30, 240, 2500)),
    ("f32", 8, 12, (14, 16, 18.5), (4, 11, 21, 30, 240, 2500)),
    ("f32", 9, 14, (), (4, 11, 16, 30, 240, 2500)), ("f32", 7, 8, (1, 300, 2500), ())])
def test_convection_over_integrated(convection_setting, dtype, nv, nq, rule, row):
    for mb in rule:
        assert convection_setting(dtype, nv, nq, mb) == 0, mb
    for mb in row:
        assert convection_setting(dtype, nv, nq, mb) == 1, mb


@pytest.mark.parametrize("dtype,n,first,second", [
    ("f64", 3, (100, 275), (290, 2500)), ("f64", 9, (100, 275, 500, 900), (1200, 2500)),
    ("f64", 13, (100, 275, 430), (600, 2500)), ("f64", 7, (600, 900), (1200,)), ("f64", 12, (240,), (290, 2500)),
    ("f32", 12, (30, 290, 500, 600), (800, 2500)), ("f32", 3, (240,), (290, 2500))])
def test_transform(dtype, n, first, second):
    fn = tpo.lib().tpo_internal_transform_setting
    fn.argtypes = [ctypes.c_int] * 2 + [ctypes.c_longlong]
    code, word = DT[dtype]
    for line, sizes in ((0, first), (1, second)):
        for mb in sizes:
            assert fn(n, code, int(mb * 1e6 / (2 * n ** 3 * word))) == line, mb
