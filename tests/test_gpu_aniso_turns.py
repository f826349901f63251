"""GPU parity of the anisotropic kernel whose passes run in turns, and of the one-turn kernel with streaming hints, against plain fp64 products on the device and the
CPU oracle: in every register class the shape with the most turns in a pass, one with the fewest elements per workgroup and
one with the most, on the smallest batch that takes it, which leaves a ragged last workgroup.  Each case asks the
library that the call takes that kernel.  Bars as for the anisotropic operator: six sums of at most 16 terms."""
import ctypes
import itertools

import numpy as np
import pytest
import torch

import oracle
from gpu_util import TOL, dev
from paper_2604_19906_amd import tpo
from paper_2604_19906_amd import workloads as wl

pytestmark = pytest.mark.gpu
DTYPES = {"f64": (tpo.TPO_F64, torch.float64, 8), "f32": (tpo.TPO_F32, torch.float32, 4)}


@pytest.fixture(scope="module", autouse=True)
def library():
    assert torch.cuda.is_available(), "GPU tests need a device"
    tpo.check(tpo.tpo_create(), "tpo_create")
    yield
    tpo.check(tpo.tpo_destroy(), "tpo_destroy")


def turns(dims, dtype, e):
    fn = tpo.lib().tpo_internal_aniso_turns
    fn.argtypes = [ctypes.c_int] * 4 + [ctypes.c_longlong]
    return divmod(fn(*dims, DTYPES[dtype][0], e), 1000)


def batch(dims, dtype):
    """The smallest batch that runs in turns with a ragged last workgroup (0: none of up to 260 MiB does)."""
    for mib in (32, 64, 96, 256):
        e = -(-(mib << 20) // (3 * dims[0] * dims[1] * dims[2] * DTYPES[dtype][2]))
        g = turns(dims, dtype, e)[0]
        if g:
            return e if g == 1 or e % g else e + 1
    return 0


def shapes(dtype, regs):
    found = []
    for dims in itertools.product(range(1, regs + 1), repeat=3):
        if len(set(dims)) == 1 or max(8, (max(dims) + 1) // 2 * 2) != regs:
            continue
        e = batch(dims, dtype)
        if e:
            g, lanes = turns(dims, dtype, e)
            nx, ny, nz = dims
            found.append((max(-(-g * p // lanes) for p in (ny * nz, nx * nz, nx * ny)), g, dims))
    return sorted({max(found)[2], min(found, key=lambda f: f[1])[2], max(found, key=lambda f: f[1])[2]})


def along(x, m, axis):
    x = x.movedim(axis, 3)
    return (x.reshape(-1, x.shape[3]) @ m).reshape(x.shape).movedim(3, axis)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("regs", [8, 10, 12, 14, 16])
def test_turns(dtype, regs):
    assert shapes(dtype, regs)
    for dims in shapes(dtype, regs):
        e = batch(dims, dtype)
        print(f"case turns {dtype} dims={dims} E={e} {turns(dims, dtype, e)}", flush=True)
        check(dims, dtype, e)


# fp64 kernel of one turn per pass with streaming hints: each size class, in both bands of batch sizes; the last workgroup
# holds fewer elements than the others (one per workgroup: none does)
@pytest.mark.parametrize("dims", [(7, 8, 6), (8, 7, 7), (9, 10, 8), (10, 9, 9), (11, 12, 10), (12, 11, 12), (15, 16, 14)])
@pytest.mark.parametrize("mib", [64, 200])
def test_streaming(dims, mib):
    e = (mib << 20) // (24 * dims[0] * dims[1] * dims[2]) // 12 * 12 + 1
    fn = tpo.lib().tpo_internal_aniso_streams
    fn.argtypes = [ctypes.c_int] * 4 + [ctypes.c_longlong]
    assert fn(*dims, tpo.TPO_F64, e) == 1 and turns(dims, "f64", e)[0] == 0
    print(f"case streaming dims={dims} E={e}", flush=True)
    check(dims, "f64", e)


def cached_shapes(regs, streams):
    """fp64 calls in turns on 320 or 440 MiB that store v_e without the non-temporal hint: fewest and most elements per workgroup."""
    found = []
    for dims in itertools.product(range(1, regs + 1), repeat=3):
        if max(8, (max(dims) + 1) // 2 * 2) != regs:
            continue
        e = -(-((320 if streams else 440) << 20) // (24 * dims[0] * dims[1] * dims[2]))
        g = turns(dims, "f64", e)[0]
        if g and hints(dims, e) == (streams, 1):
            found.append((g, dims, e))
    return [min(found), max(found)]


def hints(dims, e, dtype="f64"):
    """(streaming hints, stores without the hint) of a call."""
    fns = [getattr(tpo.lib(), f"tpo_internal_aniso_{k}") for k in ("streams", "caches")]
    for fn in fns:
        fn.argtypes = [ctypes.c_int] * 4 + [ctypes.c_longlong]
    return tuple(fn(*dims, DTYPES[dtype][0], e) for fn in fns)


@pytest.mark.parametrize("regs", [8, 10, 12, 14, 16])
@pytest.mark.parametrize("streams", [0, 1])
def test_cached_stores_in_turns(regs, streams):
    if (regs, streams) == (8, 1):
        return                  # no shape of this class with 128 points and such a face runs in turns
    for g, dims, e in cached_shapes(regs, streams):
        e += g > 1 and e % g == 0
        assert hints(dims, e) == (streams, 1) and turns(dims, "f64", e)[0] == g
        print(f"case cached turns dims={dims} E={e} streams={streams} g={g}", flush=True)
        check(dims, "f64", e)


@pytest.mark.parametrize("dims,dtype,mib", [((3, 3, 5), "f64", 224), ((5, 2, 2), "f64", 440), ((8, 3, 5), "f64", 224), ((6, 7, 3), "f64", 440),
                                            ((4, 3, 3), "f32", 184), ((6, 3, 3), "f32", 408), ((3, 2, 5), "f32", 184)])
def test_cached_stores_in_one_turn(dims, dtype, mib):
    e = -(-(mib << 20) // (3 * dims[0] * dims[1] * dims[2] * DTYPES[dtype][2])) + 1
    assert hints(dims, e, dtype) == (0, 1) and turns(dims, dtype, e)[0] == 0
    print(f"case cached {dtype} dims={dims} E={e}", flush=True)
    check(dims, dtype, e)


def check(dims, dtype, e):
    rng = np.random.default_rng([19906, 81, *dims])
    real = np.float64 if dtype == "f64" else np.float32
    mats = [dev(wl.orthogonal_matrix(n, rng).astype(real)) for n in dims]
    gen = torch.Generator(device="cuda").manual_seed(100 * dims[0] + 10 * dims[1] + dims[2])
    field = lambda lo, hi: torch.empty((e, *dims), device="cuda", dtype=DTYPES[dtype][1]).uniform_(lo, hi, generator=gen)
    u, d = field(-1, 1), field(0.03, 3.3)
    out = torch.full_like(u, float("nan"))
    tpo.apply_aniso_tensors(u, *mats, d, v=out)
    torch.cuda.synchronize()
    f, m64 = u.double(), [m.double() for m in mats]
    for axis in (1, 2, 3):
        f = along(f, m64[axis - 1], axis)
    f = f * d.double()
    for axis in (1, 2, 3):
        f = along(f, m64[axis - 1].t().contiguous(), axis)
    err = (out.double() - f).abs().flatten(1).max(dim=1).values / f.abs().flatten(1).max(dim=1).values
    assert float(err.max()) <= TOL[dtype]               # a NaN left in the output fails this too
    tail = slice(e - 70, e)
    ref = oracle.ihelm_apply_aniso(*(x.cpu().numpy() for x in (u[tail], *mats, d[tail])))
    assert oracle.max_rel_err_per_element(out[tail].cpu().numpy(), ref) <= TOL[dtype]
    tpo.apply_aniso_tensors(u, *mats, d, v=u)            # in place
    torch.cuda.synchronize()
    assert torch.equal(u, out)
