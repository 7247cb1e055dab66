"""The loops and forms that only larger calls reach: several right-hand sides on held links, several chunks of an
aggregate per workgroup, groups of two right-hand sides with a rest, the even-odd hop's forms inside the
smoother, and each form of a choice by size."""
import numpy as np
import pytest
import torch

import fields
from oracle import transfer
from tests._util import to_gpu, to_np, rel, banner

pytestmark = pytest.mark.gpu

# sums of about 40 products and, for the clover term, 12 more (f32: inputs rounded to 2^-24 as well)
TOL = {"f64": 1e-14, "f32": 4.8e-6, "bf16": 6e-3, "f16": 8e-4}


def _fields(dims, nrhs, seed):
    V = int(np.prod(dims))
    g = torch.Generator(device="cuda").manual_seed(seed)
    m = torch.view_as_complex(torch.randn(256, 3, 3, 2, generator=g, device="cuda", dtype=torch.float64))
    q, _ = torch.linalg.qr(m.cpu())
    q = (q / torch.linalg.det(q)[:, None, None] ** (1.0 / 3.0)).cuda()  # SU(3)
    U = q[torch.randint(0, 256, (4, V), generator=g, device="cuda")].contiguous()
    return U, torch.view_as_complex(torch.randn(nrhs, V, 4, 3, 2, generator=g, device="cuda", dtype=torch.float64))


def _rel(a, b):
    return float(torch.linalg.vector_norm(a - b) / torch.linalg.vector_norm(b))


def _canonical(qmg, lat, U, psi, prec, clov, dag):
    """Operator on canonical fields in storage type prec, widened to double."""
    if prec in ("f64", "f32"):
        t = torch.complex128 if prec == "f64" else torch.complex64
        u, p = U.to(t), psi.to(t)
    else:
        t = torch.bfloat16 if prec == "bf16" else torch.float16
        u, p = torch.view_as_real(U).to(t), torch.view_as_real(psi).to(t)
    if clov:
        r = qmg.clover_apply(lat, u, qmg.clover_field(lat, U, 0.9, 1.1, prec), p, dagger=dag)
    else:
        r = (qmg.wilson_apply_adj if dag else qmg.wilson_apply)(lat, u, p)
    return r.to(torch.complex128) if r.is_complex() else torch.view_as_complex(r.double())


def _native64(qmg, lat, U, psi, clov, dag):
    u, p = qmg.pack_gauge(lat, U), qmg.pack_spinor(lat, psi)
    if clov:
        r = qmg.clover_apply(lat, u, qmg.clover_field(lat, U, 0.9, 1.1), p, layout="native", dagger=dag)
    else:
        r = (qmg.wilson_apply_adj if dag else qmg.wilson_apply)(lat, u, p, layout="native")
    return qmg.unpack_spinor(lat, r)


# four directions: one group of right-hand sides over 2108 tiles with a remainder, two uneven groups over 900;
# one thread per site and right-hand side: sizes between, with a last tile that is not full
CANON = [((17, 16, 16, 31), 5, "f64"), ((17, 16, 16, 31), 5, "f32"), ((9, 16, 16, 25), 7, "f64"),
         ((9, 16, 16, 25), 7, "f32"), ((17, 16, 16, 31), 3, "bf16"), ((10, 10, 10, 17), 3, "f32"),
         ((5, 6, 7, 9), 12, "f32"), ((12, 11, 10, 14), 3, "f16"), ((15, 16, 13, 12), 1, "f64"), ((10, 10, 10, 16), 4, "f64")]


@pytest.mark.parametrize("dims,nrhs,prec", CANON)
@pytest.mark.parametrize("clov", [False, True])
def test_canonical_loops(qmg, dims, nrhs, prec, clov):
    banner(f"canonical loops {dims} nrhs={nrhs} {prec} clover={clov}")
    U, psi = _fields(dims, nrhs, 11)
    lat = qmg.Lattice(dims, 0.1, 2.0, -1)
    for dag in (False, True):
        got = _canonical(qmg, lat, U, psi, prec, clov, dag)
        ref = _native64(qmg, lat, U, psi, clov, dag)
        for r in range(nrhs):
            assert _rel(got[r], ref[r]) < TOL[prec], (r, dag)


@pytest.mark.parametrize("dims,nrhs,clov", [((16, 16, 16, 32), 9, True), ((4, 16, 32, 64), 9, True), ((2, 33, 32, 32), 2, False),
                                            ((2, 17, 32, 33), 30, True)])
@pytest.mark.parametrize("dag", [False, True])
def test_pair_groups_with_a_rest(qmg, dims, nrhs, clov, dag):
    banner(f"pairs, groups of two and a rest {dims} nrhs={nrhs} clover={clov} dag={dag}")
    U, psi = _fields(dims, nrhs, 12)
    lat = qmg.Lattice(dims, 0.1, 2.0, -1)
    A = qmg.clover_field(lat, U, 0.9, 1.1, "f32") if clov else None
    u, p = qmg.pack_gauge(lat, U, "f32"), qmg.pack_spinor(lat, psi, "f32")
    if clov:
        d = qmg.clover_apply(lat, u, A, p, layout="native", dagger=dag)
    else:
        d = (qmg.wilson_apply_adj if dag else qmg.wilson_apply)(lat, u, p, layout="native")
    d = qmg.unpack_spinor(lat, d, "f32")
    ref = _native64(qmg, lat, U, psi, clov, dag)
    for r in range(nrhs):
        assert _rel(d[r], ref[r]) < TOL["f32"], r
    if any(L % 2 for L in dims):
        return
    out = {}
    for prec in ("f32", "f64"):
        Ae, Ai = qmg.eo_site_term(lat, U, 0.9, 1.1, prec) if clov else (None, None)
        e, _ = qmg.eo_pack_spinor(lat, psi, prec)
        out[prec] = qmg.schur_apply(lat, qmg.eo_pack_gauge(lat, U, prec), e, Ae, Ai, dagger=dag).to(torch.complex128)
    for r in range(nrhs):
        assert _rel(out["f32"][r], out["f64"][r]) < 2 * TOL["f32"], r


# The smoother's source and reconstruction hops: one step of the outer solver with two sites per thread against the
# same step with one (single precision both; what their roundings make of a few Krylov steps stays far below the
# step that a wrong hop would make)
@pytest.mark.parametrize("nrhs", [1, 5])
@pytest.mark.parametrize("clov", [False, True])
@pytest.mark.parametrize("sstep", [False, True])
def test_pair_hops_in_the_smoother(qmg, nrhs, clov, sstep):
    dims = (16, 16, 32, 32)
    banner(f"pair hops in the smoother {dims} nrhs={nrhs} clover={clov} sstep={sstep}")
    U, b = _fields(dims, nrhs, 13)
    U = fields_near_one(U)
    lat = qmg.Lattice(dims, 0.1, 1.0, -1)
    mg = qmg.mg_setup_stream_chiral_svd(lat, U, (4, 4, 4, 4), 8, 4, 4, n_setup_iter=4, inner="f32", seed=3,
                                        c_sw=1.0 if clov else None)
    mg.set_smoother(eo=True, sstep=sstep)
    x = {}
    try:
        for v in (0, 1):
            qmg.set_dslash_variant(v)
            x[v], _ = qmg.mg_solve(mg, b, tol=1e-14, max_outer=1, check=False)
    finally:
        qmg.set_dslash_variant(0)
    mg.close()
    assert _rel(x[0], b) > 0.1
    for r in range(nrhs):
        assert _rel(x[0][r], x[1][r]) < 1e-3, r


def fields_near_one(U):
    """Links between one and U, projected back: U -> (1 + 0.3 U), orthonormal rows, determinant one."""
    m = torch.eye(3, dtype=U.dtype, device=U.device) + 0.3 * U
    r0 = m[..., 0, :] / torch.linalg.vector_norm(m[..., 0, :], dim=-1, keepdim=True)
    r1 = m[..., 1, :] - (r0.conj() * m[..., 1, :]).sum(-1, keepdim=True) * r0
    r1 = r1 / torch.linalg.vector_norm(r1, dim=-1, keepdim=True)
    r2 = torch.linalg.cross(r0, r1).conj()
    return torch.stack([r0, r1, r2], -2).contiguous()


# 768 aggregates of 256 sites: three, three and two of eight chunks per workgroup, passes of 8 and of 16
# right-hand sides; and an LDS demand between 60 and 68 KB
@pytest.mark.parametrize("dims,block,rank,prec,counts", [((16, 16, 24, 32), (4, 4, 4, 4), 5, "f32", (2, 9)),
                                                         ((16, 16, 24, 32), (4, 4, 4, 4), 5, "f64", (2, 9)),
                                                         ((4, 8, 4, 4), (4, 4, 4, 2), 32, "f64", (6, 15))])
def test_transfer_loops(qmg, dims, block, rank, prec, counts):
    banner(f"transfer loops {dims} block {block} rank {rank} {prec}")
    lat = qmg.Lattice(dims, 0.1, 1.0, -1)
    U, _ = _fields(dims, 1, 14)
    mg = qmg.mg_setup_stream_chiral_svd(lat, U, block, rank, rank, rank, n_setup_iter=0, inner=prec, seed=3)
    P = to_np(mg.prolongator()[0])
    t = torch.complex128 if prec == "f64" else torch.complex64
    if prec == "f32":
        P = P.astype(np.complex64).astype(np.complex128)
    tol = {"f64": 1.2e-14, "f32": 6e-6}[prec]  # sums of up to 6 * 256 products in chains of at most 48
    for nrhs in counts:
        psi = _fields(dims, nrhs, 15)[1].to(t)
        vc = to_gpu(fields.gaussian_coarse(mg.n_agg * 2 * rank, nrhs, 23).reshape(nrhs, mg.n_agg, 2, rank)).to(t)
        ref_c = transfer.restrict(P, to_np(psi).astype(np.complex128), dims, block)
        ref_f = transfer.prolong(P, to_np(vc).astype(np.complex128), dims, block)
        assert rel(to_np(qmg.restrict(mg, psi)).reshape(-1), np.asarray(ref_c).reshape(-1)) < tol, nrhs
        assert rel(to_np(qmg.prolong(mg, vc)).reshape(-1), np.asarray(ref_f).reshape(-1)) < tol, nrhs
    mg.close()


# ranks between the tiles on either side of the choice: 64 and 256 aggregates
@pytest.mark.parametrize("dims", [(4, 4, 8, 8), (8, 8, 8, 8)])
@pytest.mark.parametrize("rank", [10, 18, 20, 24])
@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_coarse_choices(qmg, dims, rank, prec):
    banner(f"coarse operator, choices {dims} rank {rank} {prec}")
    lat = qmg.Lattice(dims, 0.1, 1.0, -1)
    U, _ = _fields(dims, 1, 16)
    mg = qmg.mg_setup_stream_chiral_svd(lat, U, (2, 2, 2, 2), rank, rank, rank, n_setup_iter=0, inner=prec, seed=3)
    t = torch.complex128 if prec == "f64" else torch.complex64
    tol = {"f64": 1.2e-14, "f32": 6e-6}[prec]  # below 100 roundings, of either side
    v = to_gpu(fields.gaussian_coarse(mg.n_agg * 2 * rank, 17, 24).reshape(17, mg.n_agg, 2, rank)).to(t)
    one = torch.cat([qmg.coarse_apply(mg, v[i:i + 1]) for i in range(17)])
    for nrhs in (3, 4, 5, 16, 17):
        assert _rel(qmg.coarse_apply(mg, v[:nrhs].contiguous()), one[:nrhs]) < 2 * tol, nrhs
    mg.close()
