"""The fp32 transform halves whose products run on the matrix cores: every n that has them, at
batches on both sides of the size where n = 8 .. 11 change form, with ragged last workgroups, against
the CPU oracle.  Both forms add in the same order, so the change of form must not show: the results
of a batch are the same bits as those of its parts."""
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


@pytest.mark.parametrize("direction", [tpo.TPO_FORWARD, tpo.TPO_BACKWARD])
@pytest.mark.parametrize("n", range(8, 17))
def test_matrix_core_transforms(n, direction):
    w = wl.custom(n, 401, "f32", key=1500 + n)
    sx, sy, sz = wl.direction_matrices(w)
    u = wl.field_u(w)
    ref = (oracle.forward if direction == tpo.TPO_FORWARD else oracle.backward)(u, sx, sy, sz)
    ts = list(map(dev, (sx, sy, sz)))
    for e in (1, 2, 5, 64, 401):
        print(f"case transform n={n} direction={direction} E={e}", flush=True)
        tu = dev(u[:e])
        out = torch.full_like(tu, float("nan"))
        tpo.transform_tensors(tu, *ts, direction, t=out)
        torch.cuda.synchronize()
        assert oracle.max_rel_err_per_element(out.cpu().numpy(), ref[:e]) <= TOL["f32"]


@pytest.mark.parametrize("n", [8, 9, 10, 11])
def test_change_of_form_at_the_cache_size(n):
    most = (256 << 20) // (8 * n ** 3)
    g = torch.Generator(device="cuda").manual_seed(n)
    u = torch.empty((most + 1, n, n, n), device="cuda").uniform_(-1, 1, generator=g)
    s = [dev(m) for m in wl.direction_matrices(wl.custom(n, 1, "f32", key=1600 + n))]
    for direction in (tpo.TPO_FORWARD, tpo.TPO_BACKWARD):
        large = tpo.transform_tensors(u, *s, direction)
        cached = tpo.transform_tensors(u[:most], *s, direction)
        torch.cuda.synchronize()
        assert torch.equal(large[:most], cached)
    ref = oracle.backward(u[-40:].cpu().numpy(), *(x.cpu().numpy() for x in s))
    assert oracle.max_rel_err_per_element(large[-40:].cpu().numpy(), ref) <= TOL["f32"]
