"""The box of the positions over the accumulator's slots: workgroup b of 256 particles adds to
slot b mod 64, so the sizes here leave slots empty, fill each once, and wrap around.  Minima and
maxima are exact, so the geometry equals the plain float64 formula bit for bit."""
import pytest
import torch

import paper_2208_02382_amd as pic
import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 256, 257, 64 * 256, 64 * 256 + 1, 200_003])
def test_box_over_the_slots(n):
    cfg = workloads.SMALL
    b = pic.Beam(n, cfg.qm_qeeV, cfg.charge_C, cfg.kin_energy_MeV, cfg.mass_MeV, cfg.shape,
                 cfg.nodes)
    for rep in range(2):  # the second reduction starts from what the first one left
        g = torch.Generator().manual_seed(100 * n + rep)
        X = torch.randn((6, n), generator=g, dtype=torch.float64) * (1e-3 if rep else 3e-3)
        b.X.copy_(X)
        b.deposit()
        origin, h, h_rest = b.geometry()
        gamma = 1.0 + cfg.kin_energy_MeV / cfg.mass_MeV
        for a in range(3):
            lo, hi = float(X[2 * a].min()), float(X[2 * a].max())
            ha = (hi - lo) / (cfg.nodes[a] - 3.5)
            assert h[a] == ha and origin[a] == lo - 1.25 * ha
            assert h_rest[a] == (gamma * ha if a == 2 else ha)
    b.close()


@pytest.mark.parametrize("n", [2, 64 * 256, 64 * 256 + 1, 300_007])
def test_geometry_from_the_prologues_last_workgroup(n):
    """A one-step call's geometry comes from the last workgroup of its first pass: the box of
    x + l px after the first half map (one rounding of the product, one of the sum, a third for
    the difference of the extremes: within 4 ulp of the largest coordinate)."""
    cfg = workloads.SMALL
    b = pic.Beam(n, cfg.qm_qeeV, cfg.charge_C, cfg.kin_energy_MeV, cfg.mass_MeV, cfg.shape,
                 cfg.nodes)
    gamma = 1.0 + cfg.kin_energy_MeV / cfg.mass_MeV
    for rep in range(2):
        g = torch.Generator().manual_seed(7 * n + rep)
        X = torch.randn((6, n), generator=g, dtype=torch.float64) * (1e-3 if rep else 2e-3)
        b.X.copy_(X)
        b.track([(0.0, 0.5)], 1)
        origin, h, _ = b.geometry()
        for a in range(3):
            l = 0.25 if a < 2 else 0.25 / gamma ** 2
            p = X[2 * a] + l * X[2 * a + 1]
            lo, hi = float(p.min()), float(p.max())
            ulp = 4 * 2.0 ** -52 * max(abs(lo), abs(hi), float((l * X[2 * a + 1]).abs().max()))
            assert abs(h[a] * (cfg.nodes[a] - 3.5) - (hi - lo)) <= ulp
            assert abs(origin[a] + 1.25 * h[a] - lo) <= ulp
    b.close()
