"""Every line length of the register transforms along every axis (the half-length real transform
along x, the padded ones along y and z, the even and odd kernel spectra), and the lengths of the
runtime-length engine beside them, against the oracle: potential and direct field in one call.
The reverse sweep's solve (source on the ghost nodes) on a few mixed grids.  Bars as for the
other grids: 1e-12 of the largest value in float64, 1e-5 with the float32 grid."""
import numpy as np
import pytest
import torch

import workloads
from oracle import adjoint as oadj
from oracle import pic as opic

pytestmark = pytest.mark.gpu

LENGTHS = (16, 18, 24, 27, 32, 36, 48, 54, 64, 72, 81, 96, 108, 128)
GRIDS = [tuple(n if a == axis else (16, 18, 24)[a] for a in range(3))
         for axis in range(3) for n in LENGTHS]
# runtime-length axes beside register ones: 2 n = 24, 18, 324, 8, 486 and n = 162, 4
GRIDS += [(12, 16, 9), (162, 18, 16), (16, 4, 243), (4, 162, 18)]


def _rel(a, b):
    return np.abs(a - b).max() / np.abs(b).max()


@pytest.mark.parametrize("nodes", GRIDS, ids=lambda g: "%dx%dx%d" % g)
def test_solve_at_every_line_length(nodes):
    import paper_2208_02382_amd as lib
    cfg = workloads.SMALL
    n = 2000
    xi = workloads.draw_xi(cfg, n=n)
    prob = opic.make_problem(n, cfg.qm_qeeV, cfg.charge_C, cfg.kin_energy_MeV, cfg.mass_MeV,
                             nodes, 1, direct_field=True)
    X = opic.init_from_normals(cfg.sigma_matrix, xi)
    geom = opic.geometry(X, prob)
    Q = opic.deposit(X, geom, prob)
    phi_o = opic.solve(Q, opic.green(geom, prob))
    E_o = opic.solve_field(Q, opic.green_field(geom, prob))
    for fp32 in (False, True):
        tol = 1e-5 if fp32 else 1e-12
        b = lib.Beam(n, cfg.qm_qeeV, cfg.charge_C, cfg.kin_energy_MeV, cfg.mass_MeV, 1, nodes,
                     grid_fp32=fp32, direct_field=True)
        b.init_from_normals(cfg.sigma_matrix, torch.from_numpy(xi).cuda())
        phi, E = b.poisson_solve(b.deposit(), phi=b.new_phi())
        assert _rel(phi.cpu().numpy(), phi_o) < tol
        for c in range(3):
            assert _rel(E[c].cpu().numpy(), E_o[c]) < tol, c
        b.close()


@pytest.mark.parametrize("nodes", [(27, 32, 36), (48, 54, 16), (64, 24, 72), (18, 81, 12)],
                         ids=lambda g: "%dx%dx%d" % g)
def test_reverse_sweep_on_mixed_lengths(nodes):
    import paper_2208_02382_amd as lib
    cfg = workloads.SMALL
    n, w = 1500, np.array([0.7, -0.4, 1.3, 0.9])
    lat = ((1.0, 0.5), (-1.0, 0.5))
    xi = workloads.draw_xi(cfg, n=n, seed=11)
    b = lib.Beam(n, cfg.qm_qeeV, cfg.charge_C, cfg.kin_energy_MeV, cfg.mass_MeV, 1, nodes)
    xi_d = torch.from_numpy(xi).cuda()
    b.init_from_normals(cfg.sigma_matrix, xi_d)
    _, dk, lam, _ = b.track_adjoint(lat, 2, w, ckpt_every=2, xi=xi_d)
    prob = opic.make_problem(n, cfg.qm_qeeV, cfg.charge_C, cfg.kin_energy_MeV, cfg.mass_MeV,
                             nodes, 1)
    _, dk_o, lam_o, _ = oadj.adjoint(opic.init_from_normals(cfg.sigma_matrix, xi),
                                     np.array([1.0, -1.0]), np.array([0.5, 0.5]), 2, prob, w)
    assert _rel(np.array(dk), dk_o) < 1e-12
    lg = lam.cpu().numpy()
    for r in range(6):
        assert _rel(lg[r], lam_o[r]) < 1e-12, r
    b.close()
