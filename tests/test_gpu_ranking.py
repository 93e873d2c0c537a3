"""The ranking of the binned deposit at the edges of its forms: the size where the particles per
thread change (2^17), one particle more than a workgroup holds, and a tile whose ranks do
not fit the packed key words (more than 2^20 particles with 4096 tiles), which is ranked anew.
The charge grid is an exact sum, so it does not depend on the tiles beyond the rounding of the
fixed-point contributions (below 1e-13 of a macroparticle's charge each)."""
import pytest
import torch

import paper_2208_02382_amd as pic
import workloads

pytestmark = pytest.mark.gpu


def _rho(X, tile):
    cfg = workloads.SMALL
    n = X.shape[1]
    b = pic.Beam(n, cfg.qm_qeeV, cfg.charge_C, cfg.kin_energy_MeV, cfg.mass_MeV, 1, (16, 16, 16),
                 tuning={"tile": tile})
    b.X.copy_(X)
    rho = [b.deposit().clone() for _ in range(2)]
    assert b.check() == pic.PIC_OK
    b.close()
    assert torch.equal(rho[0], rho[1])
    return rho[0]


@pytest.mark.parametrize("n,core", [(257, 1.0), (1 << 17, 1.0), ((1 << 17) + 1, 1.0),
                                    (1 << 20, 1.0), ((1 << 20) + 1, 1.0),
                                    ((1 << 20) + 70_001, 1e-3)])
def test_ranking_forms_give_the_same_charge(n, core):
    g = torch.Generator(device="cuda").manual_seed(n)
    X = 1e-3 * core * torch.randn((6, n), generator=g, dtype=torch.float64, device="cuda")
    X[:, 0], X[:, n - 1] = -6e-3, 6.1e-3  # the box; with core 1e-3 all others share one tile
    ref = _rho(X, (16, 16, 16))
    rho = _rho(X, (1, 1, 1))
    # every contribution of the two grids is rounded within 2^-51 of the macro charge, and at
    # most n of them meet at a node (8 stencil nodes each)
    bar = 2.0 * n * 2.0 ** -51 * workloads.SMALL.charge_C / n * 8
    assert float((rho - ref).abs().max()) <= bar
    assert abs(float(rho.sum()) + workloads.SMALL.charge_C) <= 1e-12 * workloads.SMALL.charge_C
