"""The reverse sweep's geometry terms, summed over the spectra, at every z line length of the
register transforms and at lengths without one (which form the convolutions), against the oracle.
One step, so that nothing but the step's own terms enters; the particles at the box's faces carry
the geometry terms, and are the largest entries of their rows.

Bars: 1e-12 of a row's largest entry in float64 (the transforms' error, a few rounding errors per
stage of at most 8 stages per axis, relative to the norm of the sums).  With the float32 grid the
strength's gradient at its bar of 1e-4; no bar is stated for its coordinate gradients, whose z rows
differ by 2e-4 on the thinnest cells here, summed over the spectra (2.06e-4 at 162x9x16) as by
convolutions (2.13e-4)."""
import numpy as np
import pytest
import torch

import workloads
from oracle import adjoint as oadj
from oracle import pic as opic

pytestmark = pytest.mark.gpu

W4 = np.array([0.7, -0.4, 1.3, 0.9])
GRIDS = [(16, 18, n) for n in (16, 18, 24, 27, 32, 36, 48, 54, 64, 72, 81, 96, 108, 128)]
GRIDS += [(16, 18, 8), (16, 18, 6), (18, 16, 162), (162, 9, 16), (12, 162, 24)]


@pytest.mark.parametrize("nodes", GRIDS, ids=lambda g: "%dx%dx%d" % g)
def test_geometry_terms_at_every_line_length(nodes):
    import paper_2208_02382_amd as lib
    cfg = workloads.SMALL
    n = 1500
    xi = workloads.draw_xi(cfg, n=n, seed=5)
    prob = opic.make_problem(n, cfg.qm_qeeV, cfg.charge_C, cfg.kin_energy_MeV, cfg.mass_MeV,
                             nodes, 1)
    X0 = opic.init_from_normals(cfg.sigma_matrix, xi)
    _, dk_o, lam_o, _ = oadj.adjoint(X0, np.array([1.0]), np.array([0.5]), 1, prob, W4)
    for fp32, bar in ((False, 1e-12), (True, 1e-4)):
        b = lib.Beam(n, cfg.qm_qeeV, cfg.charge_C, cfg.kin_energy_MeV, cfg.mass_MeV, 1, nodes,
                     grid_fp32=fp32)
        b.init_from_normals(cfg.sigma_matrix, torch.from_numpy(xi).cuda())
        _, dk, lam, _ = b.track_adjoint(((1.0, 0.5),), 1, W4, ckpt_every=1)
        b.close()
        assert np.abs(np.array(dk) - dk_o).max() <= bar * np.abs(dk_o).max()
        if fp32:
            continue
        lg = lam.cpu().numpy()
        for r in range(6):
            scale = np.abs(lam_o[r]).max()
            assert np.abs(lg[r] - lam_o[r]).max() <= bar * scale
