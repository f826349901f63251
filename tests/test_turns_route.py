"""Which anisotropic calls run their passes in turns, asked of the library on the host: the shapes and batches on
which that is the faster form, and that what it then launches fits the kernel."""
import ctypes
import itertools

import pytest

from paper_2604_19906_amd import tpo


@pytest.fixture(scope="module")
def turns():
    fn = tpo.lib().tpo_internal_aniso_turns
    fn.argtypes = [ctypes.c_int] * 4 + [ctypes.c_longlong]
    return lambda dims, dtype, e: divmod(fn(*dims, dtype, e), 1000)


def elems(dims, dtype, megabytes):
    word = 8 if dtype == tpo.TPO_F64 else 4
    return int(megabytes * 1e6 / (3 * dims[0] * dims[1] * dims[2] * word))


# time in turns over the time in one turn per pass on MI355X beside each
@pytest.mark.parametrize("dims,dtype,mb,taken", [
    ((3, 9, 16), tpo.TPO_F64, 800, True),       # 0.47
    ((16, 9, 3), tpo.TPO_F64, 100, True),       # 0.71
    ((12, 16, 6), tpo.TPO_F64, 800, True),      # 0.83
    ((12, 16, 6), tpo.TPO_F64, 100, False),     # 0.93 .. 1.00
    ((4, 6, 15), tpo.TPO_F64, 40, False),       # 1.14
    ((4, 14, 7), tpo.TPO_F64, 20, False),       # 1.12
    ((11, 6, 5), tpo.TPO_F64, 800, False),      # 1.05
    ((14, 4, 4), tpo.TPO_F64, 100, False),      # 1.05
    ((14, 4, 4), tpo.TPO_F64, 300, True),       # 0.92
    ((3, 12, 3), tpo.TPO_F64, 300, False),      # 1.08
    ((12, 3, 3), tpo.TPO_F32, 800, False),      # 1.07
    ((5, 9, 3), tpo.TPO_F64, 800, False),       # 1.03
    ((11, 11, 14), tpo.TPO_F64, 3000, False),   # 1.14
    ((3, 9, 15), tpo.TPO_F32, 800, True),       # 0.42
    ((14, 4, 3), tpo.TPO_F32, 100, True),       # 0.79
    ((14, 4, 3), tpo.TPO_F32, 40, True),        # 0.8
    ((16, 7, 6), tpo.TPO_F32, 20, False),
    ((12, 12, 16), tpo.TPO_F32, 3000, False),   # the slice kernel's
])
def test_lines(turns, dims, dtype, mb, taken):
    assert (turns(dims, dtype, elems(dims, dtype, mb))[0] > 0) == taken


# Calls whose result is stored without the non-temporal hint; time with the hint gone over with it beside each
F64, F32 = tpo.TPO_F64, tpo.TPO_F32


@pytest.mark.parametrize("dims,dtype,mb,taken", [
    ((13, 3, 3), F64, 480, True),        # 0.83, in turns, u_e not streamed
    ((13, 3, 3), F64, 400, False),       # 0.95 there on the same fields, 1.11 on (13,1,9), 1.14 on (8,1,14)
    ((16, 3, 3), F64, 350, True),        # 0.90, u_e streamed
    ((16, 3, 3), F64, 600, True),        # 1.02 on the same fields, 0.91 on three sets in turn
    ((16, 3, 3), F64, 300, False),       # 1.02 .. 1.07 on (11,4,3), (16,12,1), (15,9,2)
    ((12, 12, 1), F64, 400, True),       # 0.96
    ((12, 12, 1), F64, 600, False),      # 1.08 on the same fields, 0.96 on three sets in turn
    ((9, 10, 2), F64, 700, False),       # 1.11 on the same fields
    ((10, 7, 2), F64, 700, False),       # 1.08 on the same fields
    ((10, 7, 2), F64, 1000, True),       # 0.92
    ((13, 1, 15), F64, 2400, True),      # 0.81
    ((16, 5, 3), F64, 700, True),        # 0.98
    ((10, 8, 2), F64, 700, False),       # 1.03: faces of whole lines
    ((9, 12, 2), F64, 700, False),       # 1.03
    ((3, 3, 5), F64, 250, True),         # 0.95, one turn per pass
    ((3, 3, 5), F64, 200, False),
    ((5, 2, 2), F64, 300, False),        # 1.25 on the same fields
    ((6, 3, 5), F64, 400, False),        # 1.24 on the same fields
    ((6, 3, 5), F64, 500, True),         # 0.96
    ((3, 4, 4), F64, 400, False),        # 1.03: lines shared by whole faces
    ((2, 7, 2), F64, 400, False),        # 1.02
    ((11, 4, 2), F64, 700, False),      # 1.01
    ((6, 3, 3), F32, 700, True),        # 0.88
    ((6, 3, 3), F32, 200, True),        # 0.85
    ((6, 3, 3), F32, 120, False),       # 1.25
    ((6, 3, 3), F32, 300, False),       # 1.38 on the same fields
    ((6, 3, 3), F32, 440, True),        # 0.89
    ((4, 3, 3), F32, 1500, True),       # 0.87
    ((4, 6, 2), F32, 400, False),       # 1.02
    ((13, 3, 3), F32, 700, False)])
def test_cached_stores(dims, dtype, mb, taken):
    fn = tpo.lib().tpo_internal_aniso_caches
    fn.argtypes = [ctypes.c_int] * 4 + [ctypes.c_longlong]
    assert fn(*dims, dtype, elems(dims, dtype, mb)) == taken


@pytest.mark.parametrize("dtype,word", [(tpo.TPO_F64, 8), (tpo.TPO_F32, 4)])
def test_what_is_launched_fits(turns, dtype, word):
    """Words per lane within the register class, LDS within 48 KB, whole wavefronts, quotients exact."""
    reached = set()
    for dims in itertools.product(range(1, 17), repeat=3):
        if len(set(dims)) == 1:
            continue
        g, lanes = turns(dims, dtype, elems(dims, dtype, 1000))
        if g == 0:
            continue
        nx, ny, nz = dims
        regs = max(8, (max(dims) + 1) // 2 * 2)
        reached.add(regs)
        assert lanes in (64, 128, 192, 256) and 1 <= g <= 64
        assert -(-g * ny * nz // lanes) * nx <= regs and -(-g * nx * ny // lanes) * nz <= regs
        assert g * nx * ((ny * (nz | 1)) | 1) * word <= 48 * 1024
        for d in {ny * nz, nx * nz, nx * ny, ny, nz} - {1}:
            inverse = -(-(1 << 23) // d)        # 24-bit product with t << 9, upper half
            most = g * max(ny * nz, nx * nz, nx * ny) - 1
            assert most << 9 < 1 << 24 and inverse < 1 << 24
            assert all(((t << 9) * inverse) >> 32 == t // d for t in {0, 1, d - 1, d, most - most % d, most - most % d - 1, most} if 0 <= t <= most)
    assert reached == {8, 10, 12, 14, 16}
