"""The coarse operator on several right-hand sides in the forms that rank, number of aggregates and of
right-hand sides choose between (row tiles of 16, passes of 8 and 16 right-hand sides, one to five groups
of wavefronts), full against the oracle with the same blocks, even-odd against one right-hand side at a
time."""
import pytest
import torch

import fields
from oracle import coarse, geometry as geo
from tests._util import to_gpu, to_np, rel, banner

pytestmark = pytest.mark.gpu

# chains of at most 16 steps of four products and nine slots: below 100 roundings (and, in FP32, that of Y)
TOL = {"f64": 1.2e-14, "f32": 6e-6}

# 16, 128 and 2048 aggregates of 2^4 sites; ranks at and beside multiples of the tiles of 16 rows
CASES = [((4, 4, 4, 4), 17), ((4, 4, 4, 4), 32), ((8, 8, 8, 4), 1), ((8, 8, 8, 4), 5), ((8, 8, 8, 4), 16),
         ((8, 8, 8, 4), 24), ((8, 8, 8, 4), 25), ((16, 16, 16, 8), 9)]


@pytest.mark.parametrize("dims,rank", CASES)
@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_coarse_forms(qmg, dims, rank, prec):
    banner(f"coarse operator {dims} rank {rank} {prec}")
    block = (2, 2, 2, 2)
    lat = qmg.Lattice(dims, 0.1, 1.0, -1)
    U = to_gpu(fields.random_gauge(dims, 0.4, 31))
    mg = qmg.mg_setup_stream_chiral_svd(lat, U, block, rank, rank, rank, n_setup_iter=0, inner=prec, seed=3)
    t = torch.complex128 if prec == "f64" else torch.complex64
    Y, cd, d = to_np(mg.coarse_blocks()), geo.coarse_dims(dims, block), mg.n_agg
    mg.set_coarse_eo(True)
    v = fields.gaussian_coarse(d * 2 * rank, 17, 32).reshape(17, d, 2, rank)
    ref = coarse.coarse_apply(Y, v, cd)
    v = to_gpu(v).to(t)
    half = v[:, : d // 2].contiguous()
    one = torch.cat([qmg.coarse_schur_apply(mg, half[i:i + 1]) for i in range(17)])
    for nrhs in (3, 5, 8, 9, 17):
        assert rel(to_np(qmg.coarse_apply(mg, v[:nrhs])), ref[:nrhs]) < TOL[prec], nrhs
        assert rel(to_np(qmg.coarse_schur_apply(mg, half[:nrhs])), to_np(one[:nrhs])) < 2 * TOL[prec], nrhs
    mg.close()


# ranks at the edges of the tiles; blocks of 16, 36, 8 and 12 sites (whole, ragged and single-site stages,
# an extent without hops inside the block)
BUILD = [((4, 4, 4, 4), (2, 2, 2, 2), 1), ((4, 4, 4, 4), (2, 2, 2, 2), 8), ((4, 4, 4, 4), (2, 2, 2, 2), 9),
         ((6, 6, 4, 4), (3, 3, 2, 2), 16), ((6, 6, 4, 4), (3, 3, 2, 2), 17), ((4, 4, 4, 2), (2, 2, 2, 1), 24),
         ((6, 4, 4, 4), (3, 2, 2, 1), 25), ((4, 4, 4, 8), (2, 2, 2, 4), 32)]


@pytest.mark.parametrize("dims,block,rank", BUILD)
def test_coarse_build_forms(qmg, dims, block, rank):
    banner(f"coarse build {dims} block {block} rank {rank}")
    m, xi = -0.1, 2.0
    U = fields.random_gauge(dims, 0.4, 33)
    lat = qmg.Lattice(dims, m, xi, -1)
    mg = qmg.mg_setup_stream_chiral_svd(lat, to_gpu(U), block, rank, rank, rank, n_setup_iter=0, inner="f64", seed=5)
    ref = coarse.build_coarse(U, to_np(mg.prolongator()[0]), m, xi, -1, dims, block)
    # sums of at most 6 * 36 products and ten terms each: below 250 roundings, half of them of either side
    assert rel(to_np(mg.coarse_blocks()), ref) < 3e-14
    mg.close()
