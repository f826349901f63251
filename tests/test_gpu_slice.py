"""GPU parity of the fp32 slice kernel (anisotropic elements on batches large enough for it) against
the CPU oracle, at the sizes where it can go wrong: every remainder of n_y and n_z by four, the
smallest and largest n_x, even and odd n_x with and without a left-over row, elements whose size
is no multiple of 16 bytes, batches at the edges of its range and of the elements each wavefront
walks over.  Bar as for the anisotropic operator: six sums of at most 16 terms in fp32."""
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


# (dims, elements): 1024 and 12288 are the ends of the rule's two ranges; from 16384 elements on a
# wavefront takes more than one
@pytest.mark.parametrize("dims,e", [
    ((5, 14, 14), 1023), ((5, 14, 14), 1024), ((7, 10, 14), 1031), ((9, 14, 15), 1500),
    ((9, 7, 16), 1024), ((14, 5, 15), 1025), ((12, 12, 16), 12287), ((12, 12, 16), 12288),
    ((13, 13, 12), 12289), ((13, 11, 14), 12288), ((15, 8, 15), 12300), ((16, 7, 16), 12291),
    ((16, 15, 13), 12290), ((15, 15, 16), 12288), ((16, 16, 15), 12288), ((10, 10, 9), 12295),
    ((11, 9, 13), 12288), ((6, 11, 10), 16383), ((6, 11, 10), 16384), ((5, 9, 11), 24577),
    ((8, 6, 13), 65543), ((5, 13, 9), 70001)])
def test_slice_shapes(dims, e):
    u, sx, sy, sz, d = inputs(dims, e, 100 * dims[0] + 10 * dims[1] + dims[2])
    print(f"case slice dims={dims} E={e}", flush=True)
    t = list(map(dev, (u, sx, sy, sz, d)))
    out = torch.full_like(t[0], float("nan"))
    tpo.apply_aniso_tensors(*t, v=out)
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    assert not np.isnan(got).any()
    idx = np.r_[0:64, e - 64:e, np.random.default_rng(3).integers(0, e, 300)]
    ref = oracle.ihelm_apply_aniso(u[idx], sx, sy, sz, d[idx])
    assert oracle.max_rel_err_per_element(got[idx], ref) <= TOL["f32"]
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


@pytest.mark.parametrize("dims", [(12, 11, 14), (13, 13, 9), (7, 10, 15), (12, 12, 16)])
def test_slice_infinities_and_nan(dims):
    """Rows and columns past the slice must not turn an infinity into a NaN: with positive matrices
    an element with +inf in it comes out +inf everywhere, one with a NaN all NaN, the others as they
    are without them."""
    e = 12288
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
