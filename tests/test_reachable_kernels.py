"""Every kernel built into the library is launched for some batch: the template arguments in the kernels' names against the
settings that the library returns for batches of every size."""
import ctypes
import re

import pytest

from kernel_metadata import kernels
from paper_2604_19906_amd import tpo

TYPE = {"d": tpo.TPO_F64, "f": tpo.TPO_F32}
SIZES = sorted({int(1.003 ** k) for k in range(8400)})        # 1 .. 8e10 elements
RECT = [(n, q) for n in range(2, 13) for q in sorted({n + 1, n + 2, (3 * n + 1) // 2}) if q <= 16]


@pytest.fixture(scope="module")
def built():
    """Kernel's name -> the template arguments of its instantiations."""
    found = {}
    for name in kernels():
        m = re.match(r"_ZN3tpo(?:12_GLOBAL__N_1)?\d+(\w+?_kernel)I(d|f)?((?:L[ib]\d+E)+)E", name)
        if m:
            found.setdefault(m.group(1), set()).add((m.group(2) or "f", *map(int, re.findall(r"\d+", m.group(3)))))
    return found


def settings(op, n, n_q, dtype):
    fn = tpo.lib().tpo_internal_setting
    fn.argtypes = [ctypes.c_int] * 4 + [ctypes.c_longlong]
    codes = {fn(op, n, n_q, dtype, e) for e in SIZES} - {-1}
    return [(c & 255, c >> 8 & 15, c >> 12 & 1, c >> 13 & 7, c >> 16) for c in codes]


def test_operator_and_halves(built):
    pencil, mm, half, half_mm = set(), set(), set(), set()
    for n in range(1, 17):
        for t, dtype in TYPE.items():
            for sep in (0, 1):
                for g, hint, xcd, _, sb in settings(sep, n, n, dtype):
                    pencil.add((t, n, g, hint, xcd, 2 * sep, sb))
                for g, hint, xcd, _, _ in settings(2 + sep, n, n, dtype):
                    mm.add((t, n, g, hint, xcd, 2 * sep))
            for g, hint, xcd, form, sb in settings(4, n, n, dtype):
                for forward in (0, 1):
                    (half_mm if form else half).add((t, n, g, hint, xcd, forward) + (() if form else (sb,)))
    assert {k[:4] + k[5:] for k in built["ihelm_pencil_kernel"]} == pencil          # all but how D arrives
    assert built["ihelm_pencil_mm_kernel"] == mm
    assert built["transform_pencil_kernel"] == half
    assert built["transform_mm_kernel"] == half_mm


def test_convection(built):
    vector, mm, rect, large = set(), set(), set(), set()
    for t, dtype in TYPE.items():
        for n in range(1, 17):
            for g, hint, xcd, form, sb in settings(5, n, n, dtype):
                flags = (form >> 1 & 1, form >> 2 & 1)
                (mm if form & 1 else vector).add((t, n, g, hint, xcd, *flags) + (() if form & 1 else (sb,)))
        for n, q in RECT:
            for g, hint, xcd, form, sb in settings(5, n, q, dtype):
                if form:
                    large.add((t, n, q, g, hint, xcd, form - 1, sb))
                else:
                    rect.add((t, n, q, g, hint, xcd, sb))
    assert built["convection_pencil_kernel"] == vector
    assert built["convection_mm_kernel"] == mm
    assert built["convection_rect_kernel"] == rect
    assert built["convection_rect_large_kernel"] == large


def test_anisotropic(built):
    """Size classes by the largest of the three sizes; (hint, renumbering) with and without streaming hints (fp64, 128 points up), and
    without the hint on the stores of thin faces (in turns in fp64, in one turn small elements)."""
    both, cached = ((2, 1), (3, 0)), ((0, 1), (1, 0))
    assert built["ihelm_aniso_kernel"] == (
        {("f", c, 2, 1) for c in (4, 6, 8, 12, 16)} | {("d", 4, 2, 1), ("d", 8, 0, 1), ("f", 4, 0, 1), ("f", 6, 0, 1)}
        | {("d", c, *h) for c in (8, 10, 12, 16) for h in both})
    assert built["ihelm_aniso_turns_kernel"] == (
        {("f", c, 2, 1) for c in (8, 10, 12, 14, 16)}
        | {("d", c, *h) for c in (8, 10, 12, 14, 16) for h in both + cached if (c, h) != (8, (1, 0))})
