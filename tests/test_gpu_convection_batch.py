"""The convection term on both sides of the batch size where its launch settings change (fields that
fit the last-level cache or not): every element against plain fp64 products on the device, the last
elements against the CPU oracle, ragged last workgroups.  Both settings add in the same order, so a
batch's results are the same bits as those of its parts.  One shape per kind of setting: other units
per workgroup, lanes numbered per phase, SPLIT, the 4x4x1 form, all loads first."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import TOL
from paper_2604_19906_amd import tpo
from paper_2604_19906_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def library():
    assert torch.cuda.is_available(), "GPU tests need a device"
    tpo.check(tpo.tpo_create(), "tpo_create")
    yield
    tpo.check(tpo.tpo_destroy(), "tpo_destroy")


SHAPES = [("f64", 3, 3), ("f64", 9, 9), ("f64", 7, 7), ("f64", 10, 10), ("f64", 2, 4), ("f64", 4, 5),
          ("f64", 7, 11), ("f64", 8, 12), ("f64", 9, 14), ("f64", 11, 12), ("f64", 11, 11), ("f64", 16, 16), ("f32", 3, 3), ("f32", 5, 5),
          ("f32", 7, 7), ("f32", 11, 11), ("f32", 13, 13), ("f32", 2, 3), ("f32", 6, 9), ("f32", 8, 12), ("f32", 10, 12),
          ("f32", 11, 13), ("f32", 12, 14)]


@pytest.mark.parametrize("dtype,nv,nq", SHAPES)
def test_both_sides_of_the_cache_size(dtype, nv, nq):
    word, dt = (8, torch.float64) if dtype == "f64" else (4, torch.float32)
    most = (256 << 20) // ((10 * nq ** 3 + 3 * nv ** 3) * word)
    e = most + 2
    w = wl.conv_custom(nv, e, dtype, key=1700 + 20 * nv + nq, nq=nq)
    d, i = (torch.from_numpy(np.ascontiguousarray(m)).cuda() for m in wl.conv_matrices(w))
    g = torch.Generator(device="cuda").manual_seed(nv * 20 + nq)
    P = torch.empty((3, 3, e, nq, nq, nq), dtype=dt, device="cuda").uniform_(-1, 1, generator=g)
    M = torch.empty((e, nq, nq, nq), dtype=dt, device="cuda").uniform_(0.5, 2, generator=g)
    print(f"case convection {dtype} ({nv},{nq}) E={e}", flush=True)
    large = tpo.convection_tensors(P, M, d, i, F=torch.full((3, e, nv, nv, nv), float("nan"), dtype=dt,
                                                            device="cuda"))
    torch.cuda.synchronize()
    for n in (most, 1, 2, 5):
        part = tpo.convection_tensors(P[:, :, :n].contiguous(), M[:n].contiguous(), d, i)
        torch.cuda.synchronize()
        assert torch.equal(part, large[:, :n])
    # direction 0 is the fastest axis: matrices along (n, m, l) per direction
    d64, i64 = d.double(), i.double()
    for c in range(3):
        ref = 0
        for k in range(3):
            x = P[c, k].double() * M.double()
            for axis in (3, 2, 1):
                mat = d64 if axis == 3 - k else i64
                x = torch.matmul(x.transpose(axis, 3), mat.t().contiguous()).transpose(axis, 3)
            ref = ref + x
        err = ((large[c].double() - ref).abs().flatten(1).max(dim=1).values
               / ref.abs().flatten(1).max(dim=1).values)
        assert float(err.max()) <= TOL[dtype]
    h = lambda t: t.cpu().numpy()
    want = oracle.convection_apply(h(P[:, :, -7:].contiguous()), h(M[-7:]), h(d), h(i))
    got = h(large[:, -7:].contiguous()).reshape(21, nv, nv, nv)
    assert oracle.max_rel_err_per_element(got, want.reshape(21, nv, nv, nv)) <= TOL[dtype]
