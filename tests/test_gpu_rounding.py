"""How often the stencils round in the sums over hops and colours, against double precision on the same inputs.
The masses make the hops the whole result.

Bounds: one rounding is uniform in half a unit in the last place, so it leaves at most u / sqrt(3) of the
number as its root mean square, u = 2^-24 or 2^-53, and 0.42 u on average over the leading digits.  With
the hops alone (no diagonal term), 24 products whose eight hops are summed one by one come to 7.8e-8 (xi = 1)
and 7.2e-8 (xi = 3.5) in a simulation in numpy, 24 single additions to 1.01e-7 and 9.6e-8; the bound lies
between."""
import numpy as np
import pytest
import torch

from tests._util import banner

pytestmark = pytest.mark.gpu

HOPS = 8.8e-8


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
