"""The stencil forms that only some sizes reach: canonical-layout tiles (remainders, groups of
right-hand sides, 16-byte and unaligned fields, 16-bit storage) against the oracle, and the
two-sites-per-thread stencils against the double-precision operator."""
import numpy as np
import pytest
import torch

import fields
from oracle import wilson
from tests._util import to_gpu, to_np, rel, banner

pytestmark = pytest.mark.gpu

# a result is a sum of about 40 products: single precision to 40 roundings of 2^-24, 16-bit
# storage to the rounding of the result (2^-9, bf16; 2^-12, f16), double to 40 * 2^-53
TOL = {"f64": 1e-14, "f32": 2.4e-6, "bf16": 3e-3, "f16": 4e-4}
REAL = {"f64": torch.float64, "f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}


def _store(a, prec, shift):
    """The array in storage type prec (16-bit: trailing pairs), its first number `shift` numbers
    into its allocation; and its values in double precision."""
    t = torch.view_as_real(to_gpu(a)).to(REAL[prec])
    vals = to_np(torch.view_as_complex(t.double()))
    buf = torch.zeros(t.numel() + 2 * shift, dtype=t.dtype, device="cuda")
    buf[2 * shift:] = t.reshape(-1)
    t = buf[2 * shift:].view(t.shape)
    return (torch.view_as_complex(t) if prec in ("f64", "f32") else t), vals


@pytest.mark.parametrize("dims", [(1, 3, 2, 2), (4, 4, 4, 4), (5, 3, 7, 3), (16, 6, 5, 4), (3, 70, 1, 2)])
@pytest.mark.parametrize("prec,nrhs,shift", [("f64", 1, 0), ("f64", 5, 0), ("f32", 1, 0), ("f32", 4, 0), ("f32", 3, 1),
                                             ("bf16", 2, 0), ("f16", 1, 0), ("bf16", 3, 1)])
@pytest.mark.parametrize("dag", [False, True])
def test_canonical_forms(qmg, dims, prec, nrhs, shift, dag):
    banner(f"canonical forms {dims} {prec} nrhs={nrhs} shift={shift} dag={dag}")
    U, Uv = _store(fields.random_gauge(dims, 0.6, 91), prec, shift)
    psi, pv = _store(fields.gaussian_spinor(dims, nrhs, 92), prec, shift)
    lat = qmg.Lattice(dims, 0.07, 2.5, -1)
    out = (qmg.wilson_apply_adj if dag else qmg.wilson_apply)(lat, U, psi)
    got = to_np(out if out.is_complex() else torch.view_as_complex(out.double()))
    ref = (wilson.apply_wilson_adj if dag else wilson.apply_wilson)(Uv, pv, 0.07, 2.5, -1, dims)
    assert rel(got, ref) < TOL[prec]


# every extent even, Lx a multiple of 4, 2^18 sites x right-hand sides or more; patches of 8, 4 and 2
# planes, rows of one pair, an odd right-hand side behind groups of two
PAIRS = [((4, 16, 64, 64), 1, False), ((12, 16, 44, 34), 1, True), ((16, 16, 32, 64), 3, False),
         ((20, 22, 18, 10), 4, True), ((8, 8, 10, 12), 40, False)]


@pytest.mark.parametrize("dims,nrhs,clov", PAIRS)
@pytest.mark.parametrize("dag", [False, True])
def test_hop_pairs(qmg, dims, nrhs, clov, dag):
    banner(f"even-odd hop, two sites per thread {dims} nrhs={nrhs} clover={clov} dag={dag}")
    V = int(np.prod(dims))
    assert V * nrhs >= 1 << 18
    g = torch.Generator(device="cuda").manual_seed(7)
    m = torch.view_as_complex(torch.randn(256, 3, 3, 2, generator=g, device="cuda", dtype=torch.float64))
    q = torch.linalg.qr(m.cpu())[0].cuda()  # unitary links
    U = q[torch.randint(0, 256, (4, V), generator=g, device="cuda")].contiguous()
    psi = torch.view_as_complex(torch.randn(nrhs, V, 4, 3, 2, generator=g, device="cuda", dtype=torch.float64))
    lat = qmg.Lattice(dims, 0.1, 2.0, -1)
    out = {}
    for prec in ("f32", "f64"):
        A, Ai = qmg.eo_site_term(lat, U, 0.9, 1.1, prec) if clov else (None, None)
        e, _ = qmg.eo_pack_spinor(lat, psi, prec)
        out[prec] = to_np(qmg.schur_apply(lat, qmg.eo_pack_gauge(lat, U, prec), e, A, Ai, dagger=dag))
    assert rel(out["f32"], out["f64"]) < 4 * TOL["f32"]  # two hops and their site terms, inputs rounded to 2^-24


# Lx even, 2^17 sites x right-hand sides or more (two right-hand sides per thread from 2^20 on): rows of one
# pair, odd extents, a last tile that is not full, an odd right-hand side behind groups of two; and
# fields off 16 bytes, which take another form
DPAIRS = [((2, 63, 32, 33), 1, False), ((6, 17, 37, 36), 1, True), ((10, 9, 13, 8), 16, False),
          ((14, 16, 17, 31), 9, True), ((16, 12, 18, 30), 11, False)]


@pytest.mark.parametrize("dims,nrhs,clov", DPAIRS)
@pytest.mark.parametrize("dag", [False, True])
def test_dslash_pairs(qmg, dims, nrhs, clov, dag):
    banner(f"dslash, two sites per thread {dims} nrhs={nrhs} clover={clov} dag={dag}")
    V = int(np.prod(dims))
    assert V * nrhs >= 1 << 17
    g = torch.Generator(device="cuda").manual_seed(8)
    U = torch.view_as_complex(torch.randn(4, V, 3, 3, 2, generator=g, device="cuda", dtype=torch.float64))
    psi = torch.view_as_complex(torch.randn(nrhs, V, 4, 3, 2, generator=g, device="cuda", dtype=torch.float64))
    lat = qmg.Lattice(dims, 0.1, 2.0, -1)
    out = {}
    for prec, shift in (("f64", 0), ("f32", 0), ("f32", 1)):
        Un, p = qmg.pack_gauge(lat, U, prec), qmg.pack_spinor(lat, psi, prec)
        buf = torch.empty(p.numel() + shift, dtype=p.dtype, device="cuda")
        buf[shift:] = p.reshape(-1)
        p = buf[shift:].view(p.shape)
        if clov:
            A = qmg.clover_field(lat, U, 0.9, 1.1, prec)
            r = qmg.clover_apply(lat, Un, A, p, layout="native", dagger=dag)
        else:
            r = (qmg.wilson_apply_adj if dag else qmg.wilson_apply)(lat, Un, p, layout="native")
        out[prec, shift] = to_np(r)
    for shift in (0, 1):
        assert rel(out["f32", shift], out["f64", 0]) < 2 * TOL["f32"]  # inputs rounded to 2^-24 as well
