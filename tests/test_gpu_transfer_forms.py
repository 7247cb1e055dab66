"""Prolongation and restriction on canonical vectors in the forms that block shape, rank and number of
right-hand sides choose between (matrix-core chunks of 16 and 32 sites, one row pack per thread),
against the oracle's transfer with the same P."""
import numpy as np
import pytest
import torch

import fields
from oracle import transfer
from tests._util import to_gpu, to_np, rel, banner

pytestmark = pytest.mark.gpu

# sums of up to 6 * 256 products in chains of at most 48: 100 roundings
TOL = {"f64": 1.2e-14, "f32": 6e-6}

# 16, 32, 128 and 256 sites (matrix cores from two right-hand sides on), 36 and 8 sites (never)
CASES = [((4, 4, 4, 6), (2, 2, 2, 2), 5), ((4, 8, 4, 4), (2, 2, 2, 4), 17), ((4, 8, 4, 4), (4, 4, 4, 2), 16),
         ((8, 4, 8, 4), (4, 4, 4, 4), 25), ((6, 6, 4, 4), (3, 3, 2, 2), 8), ((4, 4, 4, 2), (2, 2, 2, 1), 6)]


@pytest.mark.parametrize("dims,block,rank", CASES)
@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_transfer_forms(qmg, dims, block, rank, prec):
    banner(f"transfers {dims} block {block} rank {rank} {prec}")
    lat = qmg.Lattice(dims, 0.1, 1.0, -1)
    U = to_gpu(fields.random_gauge(dims, 0.4, 21))
    mg = qmg.mg_setup_stream_chiral_svd(lat, U, block, rank, rank, rank, n_setup_iter=0, inner=prec, seed=3)
    P = to_np(mg.prolongator()[0])
    t = torch.complex128 if prec == "f64" else torch.complex64
    if prec == "f32":
        P = P.astype(np.complex64).astype(np.complex128)
    for nrhs in (1, 2, 8, 9, 17):
        psi = to_gpu(fields.gaussian_spinor(dims, nrhs, 22)).to(t)
        vc = to_gpu(fields.gaussian_coarse(mg.n_agg * 2 * rank, nrhs, 23).reshape(nrhs, mg.n_agg, 2, rank)).to(t)
        ref_c = transfer.restrict(P, to_np(psi).astype(np.complex128), dims, block)
        ref_f = transfer.prolong(P, to_np(vc).astype(np.complex128), dims, block)
        got_c, got_f = to_np(qmg.restrict(mg, psi)), to_np(qmg.prolong(mg, vc))
        assert rel(got_c.reshape(-1), np.asarray(ref_c).reshape(-1)) < TOL[prec], nrhs
        assert rel(got_f.reshape(-1), np.asarray(ref_f).reshape(-1)) < TOL[prec], nrhs
    mg.close()
