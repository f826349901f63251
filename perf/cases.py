"""What this library is timed on: the tensor-product operators as a program calls them, one
library call (or one pair of calls) per pass on device tensors that the program already holds.

A case is a dict of plain values:

    op      "ihelm"    v = (Sx x Sy x Sz) diag(D) (Sx x Sy x Sz)^T u, cubic elements
            "sep"      the same with the diagonal given by its eigenvalues and a shift per element
            "pair"     the two transform halves of a spectral method in one pass: forward of one
                       field, backward of another
            "forward", "backward"   one transform half
            "conv"     volume term of the convective flux (three components, three directions)
            "aniso"    "ihelm" on elements with different sizes per axis
    dtype   "f64" or "f32"
    dims    points per axis (conv: nodes and quadrature points per direction)
    elems   elements in the batch
    shared  one direction matrix for all three axes (a mesh with one order and one reference
            operator) or three of them

The listed sizes are the configurations of ``paper_2604_19906_amd.workloads`` and of
``bench.py``; ``draw`` takes every order, type, operation and batch size in between.
"""
import math

import torch

from paper_2604_19906_amd import tpo

DTYPES = {"f64": torch.float64, "f32": torch.float32}
WORD = {"f64": 8, "f32": 4}
MAX_N = 16      # points per axis the library takes


def _case(op, dtype, dims, elems, shared=False, **extra):
    return dict(op=op, dtype=dtype, nx=dims[0], ny=dims[1], nz=dims[2], elems=elems,
                shared=shared, **extra)


def listed():
    cube = lambda n: (n, n, n)
    return [
        # a small mesh, one call per solver step: the launch path counts
        dict(name="ihelm_f64_n7_E1000", **_case("ihelm", "f64", cube(7), 1000, True)),
        # the paper's batch of 8192 elements per call
        dict(name="ihelm_f64_n8_E8192", **_case("ihelm", "f64", cube(8), 8192, True)),
        # the headline workload of bench.py: a large mesh at a common order
        dict(name="ihelm_f64_n11_E262144", **_case("ihelm", "f64", cube(11), 262144, True)),
        # the highest order
        dict(name="ihelm_f64_n16_E65536", **_case("ihelm", "f64", cube(16), 65536, True)),
        # single precision with three operators: the largest batch
        dict(name="ihelm_f32_n13_E1048576", **_case("ihelm", "f32", cube(13), 1048576)),
        # fast diagonalisation without a stored diagonal
        dict(name="sep_f64_n11_E262144", **_case("sep", "f64", cube(11), 262144, True)),
        # to modal space and back, a batch that divides by nothing
        dict(name="pair_f32_n13_E262143", **_case("pair", "f32", cube(13), 262143)),
        # flux term of a flow solver in both types, and with over-integration
        dict(name="conv_f64_n11_E32768", **_case("conv", "f64", (11, 11, 11), 32768)),
        dict(name="conv_f32_n13_E65536", **_case("conv", "f32", (13, 13, 13), 65536)),
        dict(name="conv_f64_n8_q12_E32768", **_case("conv", "f64", (8, 12, 12), 32768)),
        # extruded meshes: another order along one axis
        dict(name="aniso_f64_11x11x14_E131072", **_case("aniso", "f64", (11, 11, 14), 131072)),
        dict(name="aniso_f32_12x12x16_E262144", **_case("aniso", "f32", (12, 12, 16), 262144)),
    ]


def draw(rng):
    """One more case: operation, type, order and batch size over the whole range (the batch so
    that a pass moves between 0.5 MB and 6 GB, over its logarithm)."""
    op = rng.choice(["ihelm", "ihelm", "ihelm", "sep", "sep", "forward", "backward", "conv",
                     "conv", "aniso", "aniso"])
    dtype = rng.choice(["f64", "f64", "f32"])
    shared = False
    if op == "aniso":
        dims = tuple(rng.randint(3, MAX_N) for _ in range(3))
        if len(set(dims)) == 1:
            dims = (dims[0], dims[1], dims[2] - 1)
    elif op == "conv":
        # as many quadrature points as nodes, or over-integration with one or two points more or
        # half as many again
        nv = rng.randint(3, MAX_N)
        nq = rng.choice([nv, nv, nv + 1, nv + 2, (3 * nv + 1) // 2])
        if nq != nv and (nv > 12 or nq > MAX_N):
            nq = nv
        dims = (nv, nq, nq)
    else:
        dims = (rng.randint(3, MAX_N),) * 3
        shared = rng.random() < 0.5
    case = _case(op, dtype, dims, 1, shared)
    per_elem = work(case)["bytes"]
    total = math.exp(rng.uniform(math.log(0.5e6), math.log(6e9)))
    case["elems"] = max(3, int(total / per_elem))
    return case


def work(case):
    """Each field read or written once, the sum-factorised number of operations."""
    e, w = case["elems"], WORD[case["dtype"]]
    a, b, c = case["nx"], case["ny"], case["nz"]
    pts = a * b * c
    op = case["op"]
    if op in ("ihelm", "aniso"):
        return {"bytes": 3 * pts * w * e, "flops": (4 * (a + b + c) + 1) * pts * e}
    if op == "sep":
        return {"bytes": (2 * pts + 1) * w * e, "flops": (4 * (a + b + c) + 5) * pts * e}
    if op in ("forward", "backward"):
        return {"bytes": 2 * pts * w * e, "flops": 2 * (a + b + c) * pts * e}
    if op == "pair":
        return {"bytes": 4 * pts * w * e, "flops": 4 * (a + b + c) * pts * e}
    v, q = a, c
    flops = 3 * (6 * q ** 3 * v + 6 * q ** 2 * v ** 2 + 4 * q * v ** 3 + 3 * q ** 3 + 2 * v ** 3)
    return {"bytes": (10 * q ** 3 + 3 * v ** 3) * w * e, "flops": flops * e}


def tolerance(case):
    """Rounding of up to six dependent sums of up to 16 terms.  Measured over the ranges of
    ``draw`` against ``exact`` (fp64: another order of the sums): rel up to 4.6e-16 / 1.75e-7, max
    up to 5e-15 / 3.3e-6 (the convection term, whose directions cancel); about four times that."""
    if case["dtype"] == "f64":
        return {"rel": 2e-15, "max": 3e-14}
    return {"rel": 7e-7, "max": 1.5e-5}


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _orthogonal(n, seed, k):
    """Q of a Gaussian's QR (signs of R's diagonal folded in), made on the host: an operator of
    the mesh that a program sets up once."""
    g = torch.Generator()
    g.manual_seed(1000003 * (seed + 1) + 7919 * k + n)
    q, r = torch.linalg.qr(torch.randn(n, n, generator=g, dtype=torch.float64))
    return (q * torch.sign(torch.diagonal(r))[None, :]).contiguous()


def _field(g, shape, dtype, lo=-1.0, hi=1.0):
    """Full-mantissa uniform values, drawn in the case's own type."""
    return torch.empty(shape, dtype=dtype, device="cuda").uniform_(lo, hi, generator=g)


def _flux_matrices(nv, nq):
    """Differentiation and interpolation from nq Chebyshev-Gauss to nv Chebyshev-Lobatto points."""
    xq = [-math.cos(math.pi * (2 * i + 1) / (2 * nq)) for i in range(nq)]
    xv = [-math.cos(math.pi * i / (nv - 1)) for i in range(nv)] if nv > 1 else [0.0]
    interp = torch.empty(nv, nq, dtype=torch.float64)
    deriv = torch.empty(nv, nq, dtype=torch.float64)
    for q in range(nq):
        others = [r for r in range(nq) if r != q]
        den = math.prod(xq[q] - xq[r] for r in others)
        for v, x in enumerate(xv):
            interp[v, q] = math.prod(x - xq[r] for r in others) / den
            deriv[v, q] = sum(math.prod(x - xq[r] for r in others if r != s)
                              for s in others) / den
    return deriv, interp


_created = []


def prepare(case, seed):
    """Fields, operators and output buffers on the device, as a solver holds them over its steps."""
    if not _created:
        tpo.check(tpo.tpo_create(), "tpo_create")
        _created.append(True)
    op, dt, e = case["op"], DTYPES[case["dtype"]], case["elems"]
    dims = (case["nx"], case["ny"], case["nz"])
    g = _generator(seed)
    st = {"op": op}
    if op == "conv":
        v, q = dims[0], dims[2]
        st["D_vq"], st["I_vq"] = (m.to(dt).cuda() for m in _flux_matrices(v, q))
        st["M"] = _field(g, (e, q, q, q), dt, 0.5, 2.0)
        st["P"] = _field(g, (3, 3, e, q, q, q), dt)
        st["F"] = torch.empty((3, e, v, v, v), dtype=dt, device="cuda")
        return st
    if case["shared"]:
        st["S"] = (_orthogonal(dims[0], seed, 0).to(dt).cuda(),) * 3
    else:
        st["S"] = tuple(_orthogonal(n, seed, k).to(dt).cuda() for k, n in enumerate(dims))
    st["u"] = _field(g, (e, *dims), dt)
    st["v"] = torch.empty_like(st["u"])
    if op == "pair":
        st["t"] = _field(g, (e, *dims), dt)
        st["w"] = torch.empty_like(st["u"])
    if op in ("ihelm", "aniso", "sep"):
        lam = [_field(g, (n,), torch.float64, 0.1, 10.0) for n in dims]
        if case["shared"]:
            lam = [lam[0]] * 3
        mu = _field(g, (e,), torch.float64, 0.0, 1.0)
        if op == "sep":
            st["lam"] = tuple(x.to(dt) for x in lam)
            if case["shared"]:
                st["lam"] = (st["lam"][0],) * 3
            st["mu"] = mu.to(dt)
        else:
            lam3 = lam[0][:, None, None] + lam[1][None, :, None] + lam[2][None, None, :]
            st["D"] = torch.empty_like(st["u"])
            step = max(1, (1 << 27) // lam3.numel())
            for lo in range(0, e, step):
                st["D"][lo:lo + step] = 1.0 / (lam3 + mu[lo:lo + step, None, None, None])
    return st


def run(st):
    """One pass through the binding's tensor functions."""
    op = st["op"]
    if op == "ihelm":
        return tpo.apply_tensors(st["u"], *st["S"], st["D"], v=st["v"])
    if op == "aniso":
        return tpo.apply_aniso_tensors(st["u"], *st["S"], st["D"], v=st["v"])
    if op == "sep":
        return tpo.apply_sep_tensors(st["u"], *st["S"], *st["lam"], st["mu"], v=st["v"])
    if op == "forward":
        return tpo.transform_tensors(st["u"], *st["S"], tpo.TPO_FORWARD, t=st["v"])
    if op == "backward":
        return tpo.transform_tensors(st["u"], *st["S"], tpo.TPO_BACKWARD, t=st["v"])
    if op == "pair":
        return (tpo.transform_tensors(st["u"], *st["S"], tpo.TPO_FORWARD, t=st["v"]),
                tpo.transform_tensors(st["t"], *st["S"], tpo.TPO_BACKWARD, t=st["w"]))
    return tpo.convection_tensors(st["P"], st["M"], st["D_vq"], st["I_vq"], F=st["F"])


def _along(x, mat, axis):
    """y[.., i, ..] = sum_l mat[i, l] x[.., l, ..] along one of the three cube axes of
    ``x [E, a, b, c]``: one plain matrix product."""
    x = x.transpose(axis, 3).contiguous()
    y = torch.mm(x.view(-1, x.shape[3]), mat.t().contiguous()).view(*x.shape[:3], mat.shape[0])
    return y.transpose(axis, 3).contiguous()


def _along_all(x, mats):
    for axis in (3, 2, 1):
        x = _along(x, mats[axis - 1], axis)
    return x


def exact(case, seed):
    """The same results in 64 bits from the same inputs, by plain matrix products."""
    st = prepare(case, seed)
    op, e = case["op"], case["elems"]
    f64 = torch.float64
    spans = range(0, e, max(1, (1 << 24) // (case["nx"] * case["ny"] * case["nz"])))
    step = spans.step
    if op == "conv":
        d, i = st["D_vq"].to(f64), st["I_vq"].to(f64)
        out = torch.empty(st["F"].shape, dtype=f64, device="cuda")
        for c in range(3):
            for lo in spans:
                m = st["M"][lo:lo + step].to(f64)
                # direction 0 is the fastest cube axis
                out[c, lo:lo + step] = sum(
                    _along_all(st["P"][c, k, lo:lo + step].to(f64) * m,
                               [d if axis == 3 - k else i for axis in (1, 2, 3)])
                    for k in range(3))
        return out
    fwd = [s.to(f64).t().contiguous() for s in st["S"]]
    bwd = [s.to(f64) for s in st["S"]]

    def whole(fn, *fields):
        out = torch.empty(st["u"].shape, dtype=f64, device="cuda")
        for lo in spans:
            out[lo:lo + step] = fn(*(f[lo:lo + step].to(f64) for f in fields))
        return out

    if op == "forward":
        return whole(lambda u: _along_all(u, fwd), st["u"])
    if op == "backward":
        return whole(lambda u: _along_all(u, bwd), st["u"])
    if op == "pair":
        return (whole(lambda u: _along_all(u, fwd), st["u"]),
                whole(lambda t: _along_all(t, bwd), st["t"]))
    if op == "sep":
        lx, ly, lz = (x.to(f64) for x in st["lam"])
        lam3 = lx[:, None, None] + ly[None, :, None] + lz[None, None, :]
        return whole(lambda u, mu: _along_all(
            _along_all(u, fwd) / (lam3 + mu[:, None, None, None]), bwd), st["u"], st["mu"])
    return whole(lambda u, d: _along_all(_along_all(u, fwd) * d, bwd), st["u"], st["D"])
