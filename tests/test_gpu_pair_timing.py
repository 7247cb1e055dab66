"""The two launches of an odd number of right-hand sides in groups of two are timed as one."""
import pytest
import torch

from tests._util import banner

pytestmark = pytest.mark.gpu


def test_rest_behind_groups_of_two_is_timed(qmg):
    dims, V = (16, 16, 16, 32), 16 ** 3 * 32
    banner(f"timing of the pair stencil {dims}")
    lat = qmg.Lattice(dims, 0.1, 1.0, -1)
    g = torch.Generator(device="cuda").manual_seed(2)
    U = torch.view_as_complex(torch.randn(4, 9, V, 2, generator=g, device="cuda"))
    ms = {}
    for nrhs in (8, 9):
        psi = torch.view_as_complex(torch.randn(nrhs, 12, V, 2, generator=g, device="cuda"))
        best = []
        for _ in range(20):
            qmg.timing_enable(True)
            qmg.wilson_apply(lat, U, psi, layout="native")
            r = qmg.timing_query("dslash/pair")
            assert r["launches"] == 1
            best.append(r["ms"])
        ms[nrhs] = min(best)
    qmg.timing_enable(False)
    # one right-hand side more is an eighth more work, and a launch of its own
    assert ms[9] > 1.06 * ms[8], ms
