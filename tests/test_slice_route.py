"""Which anisotropic fp32 calls take the slice kernel, asked of the library on the host: the shapes that it
is slower on stay with the runtime-size pencil kernel, and the classes it is built for are the ones
that some call reaches."""
import ctypes
import itertools

import pytest

from paper_2604_19906_amd import tpo

BATCHES = (1, 1023, 1024, 2047, 2048, 12287, 12288, 24575, 24576, 1 << 20)


@pytest.fixture(scope="module")
def takes():
    fn = tpo.lib().tpo_internal_aniso_takes_slice
    fn.argtypes = [ctypes.c_int] * 4 + [ctypes.c_longlong]
    return lambda dims, e, dtype=tpo.TPO_F32: bool(fn(*dims, dtype, e))


# time of the slice kernel over that of the pencil kernel on MI355X beside each
@pytest.mark.parametrize("dims,e", [
    ((16, 7, 9), 16534),       # 1.22
    ((13, 5, 10), 33333),      # 1.18
    ((12, 5, 11), 25252),      # 1.14
    ((13, 6, 10), 53418),      # 1.11
    ((13, 9, 13), 16436),      # 1.11
    ((16, 13, 9), 13354),      # 1.49
    ((16, 13, 10), 24038),     # 1.22
    ((15, 15, 13), 17094),     # 1.02
    ((15, 15, 16), 13888),     # 1.00
    ((14, 16, 16), 1395),      # 1.10
    ((13, 16, 16), 1502),      # 1.14
])
def test_slower_shapes_stay_with_the_pencil_kernel(takes, dims, e):
    assert not takes(dims, e)


# the same ratio where the slice kernel is ahead
@pytest.mark.parametrize("dims,e", [
    ((12, 12, 16), 262144),    # 0.74
    ((9, 5, 16), 138888),      # 0.67
    ((5, 9, 12), 185185),      # 0.69
    ((16, 16, 15), 54253),     # 0.84
    ((13, 16, 16), 6010),      # 0.82
    ((13, 5, 16), 2003),       # 0.74
    ((9, 14, 15), 1500),       # 0.64
])
def test_faster_shapes_take_the_slice_kernel(takes, dims, e):
    assert takes(dims, e)
    assert not takes(dims, e, tpo.TPO_F64)


def test_built_classes_are_the_reached_ones(takes):
    built = tpo.lib().tpo_internal_slice_class_built
    reached = set()
    for dims in itertools.product(range(1, 17), repeat=3):
        if len(set(dims)) > 1 and any(takes(dims, e) for e in BATCHES):
            reached.add((dims[0], (dims[1] + 3) // 4, (dims[2] + 3) // 4))
    assert reached == {c for c in itertools.product(range(1, 17), range(1, 5), range(1, 5)) if built(*c)}
