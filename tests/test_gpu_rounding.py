"""How often the stencils round: sums over hops and colours, and the diagonal term, in the forms that hand their
partial sums on (two sites per thread, one direction per wavefront), against double precision on the same
inputs.  The masses make the part in question the whole result.

Bounds: one rounding is uniform in half a unit in the last place, so it leaves at most u / sqrt(3) of the
number as its root mean square, u = 2^-24 or 2^-53, and 0.42 u on average over the leading digits.  With
the hops alone (no diagonal term), 24 products whose eight hops are summed one by one come to 7.8e-8 (xi = 1)
and 7.2e-8 (xi = 3.5) in a simulation in numpy, 24 single additions to 1.01e-7 and 9.6e-8; the bound lies
between.  A diagonal term of 50 times the hops leaves its own rounding; added first it would be rounded
five times (5.6e-8)."""
import numpy as np
import pytest
import torch

import fields
from oracle import wilson
from tests._util import to_gpu, to_np, rel, banner

pytestmark = pytest.mark.gpu

HOPS = 8.8e-8
ONCE = 1.05 / 3.0 ** 0.5


def _fields(dims, nrhs, seed):
    V = int(np.prod(dims))
    g = torch.Generator(device="cuda").manual_seed(seed)
    m = torch.view_as_complex(torch.randn(256, 3, 3, 2, generator=g, device="cuda", dtype=torch.float64))
    q = torch.linalg.qr(m.cpu())[0].cuda()  # unitary links
    U = q[torch.randint(0, 256, (4, V), generator=g, device="cuda")]
    psi = torch.view_as_complex(torch.randn(nrhs, V, 4, 3, 2, generator=g, device="cuda", dtype=torch.float64))
    # as single precision holds them
    return U.to(torch.complex64).to(torch.complex128).contiguous(), psi.to(torch.complex64).to(torch.complex128)


def _rel(a, b):
    return float(torch.linalg.vector_norm(a.to(torch.complex128) - b) / torch.linalg.vector_norm(b))


# one and two right-hand sides per thread
@pytest.mark.parametrize("nrhs", [9, 65])
@pytest.mark.parametrize("xi", [1.0, 3.5])
@pytest.mark.parametrize("dag", [False, True])
def test_pair_stencil_sums_whole_hops(qmg, nrhs, xi, dag):
    dims = (8, 8, 16, 16)
    banner(f"rounding of the pair stencil {dims} nrhs={nrhs} xi={xi} dag={dag}")
    U, psi = _fields(dims, nrhs, 3)
    lat = qmg.Lattice(dims, -(1.0 + 3.0 / xi), xi, -1)
    op = qmg.wilson_apply_adj if dag else qmg.wilson_apply
    out = {p: op(lat, qmg.pack_gauge(lat, U, p), qmg.pack_spinor(lat, psi, p), layout="native") for p in ("f32", "f64")}
    assert _rel(out["f32"], out["f64"]) < HOPS


@pytest.mark.parametrize("nrhs", [17, 65])
@pytest.mark.parametrize("xi", [1.0, 3.5])
@pytest.mark.parametrize("dag", [False, True])
def test_pair_hop_sums_whole_hops(qmg, nrhs, xi, dag):
    dims = (8, 8, 16, 16)
    banner(f"rounding of the even-odd pair hop {dims} nrhs={nrhs} xi={xi} dag={dag}")
    U, psi = _fields(dims, nrhs, 4)
    lat = qmg.Lattice(dims, 0.1 - (1.0 + 3.0 / xi), xi, -1)  # 0.1 x - 10 H H x
    out = {}
    for p in ("f32", "f64"):
        e, _ = qmg.eo_pack_spinor(lat, psi, p)
        out[p] = qmg.schur_apply(lat, qmg.eo_pack_gauge(lat, U, p), e, dagger=dag)
    assert _rel(out["f32"], out["f64"]) < 2.0 ** 0.5 * HOPS  # two hops


# canonical: four directions per workgroup; native: the direction split (odd rows of the lattice)
@pytest.mark.parametrize("layout", ["canonical", "native"])
@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("dag", [False, True])
def test_diagonal_term_is_rounded_once(qmg, layout, prec, dag):
    dims, m, xi = (5, 6, 4, 8), 50.5, 2.0
    banner(f"rounding of the diagonal term {dims} {prec} {layout} dag={dag}")
    U, psi = fields.random_gauge(dims, 0.6, 5), fields.gaussian_spinor(dims, 3, 6)
    t, u = (np.complex128, 2.0 ** -53) if prec == "f64" else (np.complex64, 2.0 ** -24)
    U, psi = U.astype(t).astype(np.complex128), psi.astype(t).astype(np.complex128)
    lat = qmg.Lattice(dims, m, xi, -1)
    op = qmg.wilson_apply_adj if dag else qmg.wilson_apply
    if layout == "native":
        a, b = qmg.pack_gauge(lat, to_gpu(U), prec), qmg.pack_spinor(lat, to_gpu(psi), prec)
        got = to_np(qmg.unpack_spinor(lat, op(lat, a, b, layout="native"), prec))
    else:
        got = to_np(op(lat, to_gpu(U.astype(t)), to_gpu(psi.astype(t))))
    ref = wilson.apply_wilson(U.astype(np.clongdouble), psi.astype(np.clongdouble), m, xi, -1, dims, dagger=dag)
    assert rel(got.astype(np.clongdouble), ref) < ONCE * u


# sums beyond the largest number are infinite, not undefined: hops below it, diagonal term above
@pytest.mark.parametrize("layout", ["canonical", "native"])
@pytest.mark.parametrize("prec,big", [("f64", 1e307), ("f32", 1e37)])
def test_overflow_stays_infinite(qmg, layout, prec, big):
    dims = (5, 6, 4, 8)
    banner(f"overflow of the diagonal term {dims} {prec} {layout}")
    U = fields.random_gauge(dims, 0.6, 5)
    psi = torch.full((3, int(np.prod(dims)), 4, 3), big, dtype=torch.complex128, device="cuda")
    lat = qmg.Lattice(dims, 50.5, 2.0, -1)
    if layout == "native":
        u, p = qmg.pack_gauge(lat, to_gpu(U), prec), qmg.pack_spinor(lat, psi, prec)
        got = qmg.unpack_spinor(lat, qmg.wilson_apply(lat, u, p, layout="native"), prec)
    else:
        t = torch.complex128 if prec == "f64" else torch.complex64
        got = qmg.wilson_apply(lat, to_gpu(U).to(t), psi.to(t))
    assert torch.all(got.real == float("inf")) and torch.all(torch.isfinite(got.imag))
