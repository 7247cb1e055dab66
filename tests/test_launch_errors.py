"""A launch that fails is reported by the call that made it: without a device every stencil call that passes the
argument checks ends in EHIP, whatever form its size chooses."""
import ctypes

import pytest
import torch

import paper_2505_14399_amd as q

EHIP = next(c for c, name in q.STATUS.items() if name == "EHIP")


@pytest.mark.skipif(torch.cuda.is_available(), reason="the addresses stand for device memory that is not there")
@pytest.mark.parametrize("dims,nrhs", [((4, 4, 4, 4), 1), ((16, 16, 16, 32), 1), ((16, 16, 16, 32), 9), ((32, 32, 32, 64), 3)])
@pytest.mark.parametrize("prec", ["f64", "f32", "bf16", "f16"])
@pytest.mark.parametrize("layout", [q.CANONICAL, q.NATIVE])
def test_failed_launch_is_reported(dims, nrhs, prec, layout):
    lib, P = q.load_library(), ctypes.c_void_p
    lat = q.Lattice(dims, 0.1, 1.0, -1).c()
    U, psi, out, A = P(1 << 30), P(1 << 40), P(1 << 41), P(1 << 42)
    p = q._PREC[prec]
    for fn in (lib.qmg_wilson_apply, lib.qmg_wilson_apply_adj):
        assert fn(ctypes.byref(lat), U, psi, out, nrhs, p, layout, None) == EHIP
    assert lib.qmg_clover_apply(ctypes.byref(lat), U, A, psi, out, nrhs, p, layout, 0, None) == EHIP
