"""GPU parity of the fp32 slice kernel (anisotropic elements on batches large enough for it) against
the CPU oracle, at the sizes where it can go wrong: every remainder of n_y and n_z by four, the
smallest and largest n_x, even and odd n_x with and without a left-over row, elements whose size
is no multiple of 16 bytes, batches at the edges of its range and of the elements each wavefront
walks over, every compiled class over several elements.  Each case asks the library that the call does
take the kernel.  Bar as for the anisotropic operator: six sums of at most 16 terms in fp32."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from gpu_util import TOL, dev
from paper_2604_19906_amd import tpo
from paper_2604_19906_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def library():
    assert torch.cuda.is_available(), "GPU tests need a device"
    tpo.check(tpo.tpo_create(), "tpo_create")
    yield
    tpo.check(tpo.tpo_destroy(), "tpo_destroy")


def inputs(dims, e, seed):
    rng = np.random.default_rng([19906, 78, seed])
    mats = [wl.orthogonal_matrix(n, rng).astype(np.float32) for n in dims]
    u = rng.uniform(-1, 1, (e, *dims)).astype(np.float32)
    d = rng.uniform(0.03, 3.3, (e, *dims)).astype(np.float32)
    return u, *mats, d


def takes_slice(dims, e):
    fn = tpo.lib().tpo_internal_aniso_takes_slice
    fn.argtypes = [ctypes.c_int] * 4 + [ctypes.c_longlong]
    return bool(fn(*dims, tpo.TPO_F32, e))


def device_inputs(dims, e):
    """The same distributions, drawn on the device."""
    rng = np.random.default_rng([19906, 79, *dims])
    mats = [dev(wl.orthogonal_matrix(n, rng).astype(np.float32)) for n in dims]
    g = torch.Generator(device="cuda").manual_seed(100 * dims[0] + 10 * dims[1] + dims[2])
    field = lambda lo, hi: torch.empty((e, *dims), device="cuda").uniform_(lo, hi, generator=g)
    return [field(-1, 1), *mats, field(0.03, 3.3)]


def check_shape(dims, e, t=None):
    print(f"case slice dims={dims} E={e}", flush=True)
    if t is None:
        t = list(map(dev, inputs(dims, e, 100 * dims[0] + 10 * dims[1] + dims[2])))
    out = torch.full_like(t[0], float("nan"))
    tpo.apply_aniso_tensors(*t, v=out)
    torch.cuda.synchronize()
    assert not torch.isnan(out).any()
    idx = np.r_[0:64, e - 64:e, np.random.default_rng(3).integers(0, e, 300)]
    at = torch.from_numpy(idx).cuda()
    u, d, got = (x[at].cpu().numpy() for x in (t[0], t[4], out))
    ref = oracle.ihelm_apply_aniso(u, *(x.cpu().numpy() for x in t[1:4]), d)
    assert oracle.max_rel_err_per_element(got, ref) <= TOL["f32"]
    # every element against plain fp64 products on the device (einsum per axis)
    t64 = [x.double() for x in t]
    f = torch.einsum("li,elmq->eimq", t64[1], t64[0])
    f = torch.einsum("mj,eimq->eijq", t64[2], f)
    f = torch.einsum("qk,eijq->eijk", t64[3], f) * t64[4]
    f = torch.einsum("il,elmq->eimq", t64[1], f)
    f = torch.einsum("jm,eimq->eijq", t64[2], f)
    f = torch.einsum("kq,eijq->eijk", t64[3], f)
    err = (out.double() - f).abs().flatten(1).max(dim=1).values / f.abs().flatten(1).max(dim=1).values
    assert float(err.max()) <= TOL["f32"]
    tpo.apply_aniso_tensors(*t, v=t[0])                       # in place
    torch.cuda.synchronize()
    assert torch.equal(t[0], out)


# (dims, elements): the ends of the rule's ranges (1024, for n_x >= 13 with n_y >= 9 2048, 12288, for the one-wavefront
# forms 24576); from 16384 elements on a wavefront takes e // 8192 elements, up to eight, with stores four
# slices at a time (n_x <= 12) or two, the last group of an odd n_x being one slice.
@pytest.mark.parametrize("dims,e", [
    ((5, 14, 14), 1024), ((7, 10, 14), 1031), ((9, 14, 15), 1500),
    ((9, 7, 16), 1024), ((14, 5, 15), 1025), ((13, 14, 14), 2048), ((12, 12, 16), 12287), ((12, 12, 16), 12288),
    ((13, 13, 12), 12289), ((13, 11, 14), 12288), ((15, 8, 15), 12300), ((16, 7, 16), 12291),
    ((11, 9, 13), 12288), ((6, 11, 10), 16383), ((6, 11, 10), 16384), ((5, 9, 11), 24577),
    ((7, 6, 14), 65543), ((5, 13, 9), 70001), ((9, 14, 15), 65543), ((10, 6, 16), 65539),
    ((13, 13, 12), 16387), ((13, 13, 12), 70001), ((15, 8, 15), 24579), ((16, 7, 16), 40961),
    ((15, 15, 16), 24583), ((16, 16, 15), 32771), ((16, 15, 13), 24577)])
def test_slice_shapes(dims, e):
    assert takes_slice(dims, e)
    check_shape(dims, e)


# the pencil kernel's calls next to the rule's lines give the same results
@pytest.mark.parametrize("dims,e", [((5, 14, 14), 1023), ((13, 14, 14), 2047), ((15, 15, 16), 24575),
                                    ((16, 7, 9), 16534), ((13, 13, 9), 12288)])
def test_next_to_the_lines(dims, e):
    assert not takes_slice(dims, e)
    check_shape(dims, e)


CLASSES = [(nx, ksb, ksc) for nx in range(5, 17) for ksb in (2, 3, 4) for ksc in (3, 4)]


@pytest.mark.parametrize("nx,ksb,ksc", CLASSES)
def test_every_class_walks(nx, ksb, ksc):
    """Three elements per wavefront and a ragged last walk in every compiled class, on its smallest shape
    that takes the kernel and its largest."""
    e = 24576 + 8191
    shapes = [(nx, ny, nz) for ny in range(4 * ksb - 3, 4 * ksb + 1) for nz in range(4 * ksc - 3, 4 * ksc + 1)
              if len({nx, ny, nz}) > 1 and takes_slice((nx, ny, nz), e)]
    if not shapes:
        built = tpo.lib().tpo_internal_slice_class_built
        assert not built(nx, ksb, ksc)
        return
    for dims in sorted({shapes[0], shapes[-1]}):
        check_shape(dims, e, device_inputs(dims, e))


@pytest.mark.parametrize("dims", [(12, 11, 14), (11, 9, 13), (13, 15, 9), (7, 10, 15), (12, 12, 16)])
def test_slice_infinities_and_nan(dims):
    """Rows and columns past the slice must not turn an infinity into a NaN: with positive matrices
    an element with +inf in it comes out +inf everywhere, one with a NaN all NaN, the others as they
    are without them."""
    e = 12288
    assert takes_slice(dims, e)
    u, sx, sy, sz, d = inputs(dims, e, 7)
    sx, sy, sz = np.abs(sx) + 0.1, np.abs(sy) + 0.1, np.abs(sz) + 0.1
    u = np.abs(u)
    u[3, dims[0] - 1, dims[1] - 1, dims[2] - 1] = np.inf
    u[5, 0, 0, 0] = np.inf
    u[6, 1, 2, 3] = np.nan
    d[9, 2, dims[1] - 1, 1] = np.inf
    got = tpo.apply_aniso_tensors(*map(dev, (u, sx, sy, sz, d))).cpu().numpy()
    ref = oracle.ihelm_apply_aniso(u[:16], sx, sy, sz, d[:16])
    assert np.array_equal(np.isnan(got[:16]), np.isnan(ref))
    assert np.array_equal(np.isposinf(got[:16]), np.isposinf(ref))
    assert np.isposinf(ref[3]).all() and np.isposinf(ref[5]).all() and np.isnan(ref[6]).all()
    keep = [i for i in range(16) if i not in (3, 5, 6, 9)]
    assert oracle.max_rel_err_per_element(got[keep], ref[keep]) <= TOL["f32"]


def test_slice_under_capture():
    """A captured call, replayed on new input, gives what the call gives."""
    dims, e = (12, 12, 16), 20000
    assert takes_slice(dims, e)
    t = device_inputs(dims, e)
    out = torch.empty_like(t[0])
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        tpo.apply_aniso_tensors(*t, v=out)
    for k in range(3):
        t[0].mul_(0.5 + k)
        out.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, tpo.apply_aniso_tensors(*t))
