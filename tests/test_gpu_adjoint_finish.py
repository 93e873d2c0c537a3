"""The end of a reverse step where particles lie on several faces of the box at once (few particles)
and where the particle kernels' workgroup count sits at a wavefront's edge or at its largest, against
the oracle.

Bar 1e-10 of a row's largest entry: rounding, times 1e5 for the cancellation between a face
particle's own terms and the geometry's (a beam of few particles moves its grid along with it)."""
import numpy as np
import pytest
import torch

import workloads
from oracle import adjoint as oadj
from oracle import pic as opic

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [8, 12, 40, 64 * 256, 64 * 256 + 1, 1024 * 256 + 1])
def test_end_of_a_reverse_step(n):
    import paper_2208_02382_amd as lib
    cfg = workloads.SMALL
    nodes, w4 = (12, 12, 12), np.array([0.7, -0.4, 1.3, 0.9])
    xi = np.random.default_rng(n).standard_normal((6, n))
    prob = opic.make_problem(n, cfg.qm_qeeV, cfg.charge_C, cfg.kin_energy_MeV, cfg.mass_MeV,
                             nodes, 1)
    X0 = opic.init_from_normals(cfg.sigma_matrix, xi)
    _, dk_o, lam_o, _ = oadj.adjoint(X0, np.array([1.0, -0.7]), np.array([0.5, 0.4]), 2, prob, w4)
    b = lib.Beam(n, cfg.qm_qeeV, cfg.charge_C, cfg.kin_energy_MeV, cfg.mass_MeV, 1, nodes)
    b.init_from_normals(cfg.sigma_matrix, torch.from_numpy(xi).cuda())
    _, dk, lam, _ = b.track_adjoint(((1.0, 0.5), (-0.7, 0.4)), 2, w4, ckpt_every=1)
    b.close()
    assert np.abs(np.array(dk) - dk_o).max() <= 1e-10 * np.abs(dk_o).max()
    lg = lam.cpu().numpy()
    for r in range(6):
        assert np.abs(lg[r] - lam_o[r]).max() <= 1e-10 * np.abs(lam_o[r]).max()


@pytest.mark.parametrize("n", [1 << 22, (1 << 22) + 1])
def test_consecutive_reverse_steps_on_both_sides_of_the_fork_rule(n):
    # the spectra of the next reverse step start in mid-step or at its end; three steps in one
    # segment.  The bar as above: rounding of sums over 4e6 particles (1e-13) times 1e3 for the
    # cancellation in the geometry's sums, which with many particles is the smaller factor
    import paper_2208_02382_amd as lib
    cfg = workloads.SMALL
    nodes, w4 = (12, 12, 12), np.array([0.7, -0.4, 1.3, 0.9])
    xi = np.random.default_rng(4).standard_normal((6, n))
    prob = opic.make_problem(n, cfg.qm_qeeV, cfg.charge_C, cfg.kin_energy_MeV, cfg.mass_MeV,
                             nodes, 1)
    X0 = opic.init_from_normals(cfg.sigma_matrix, xi)
    _, dk_o, lam_o, _ = oadj.adjoint(X0, np.array([1.0]), np.array([0.5]), 3, prob, w4)
    b = lib.Beam(n, cfg.qm_qeeV, cfg.charge_C, cfg.kin_energy_MeV, cfg.mass_MeV, 1, nodes)
    b.init_from_normals(cfg.sigma_matrix, torch.from_numpy(xi).cuda())
    _, dk, lam, _ = b.track_adjoint(((1.0, 0.5),), 3, w4, ckpt_every=3)
    b.close()
    assert np.abs(np.array(dk) - dk_o).max() <= 1e-10 * np.abs(dk_o).max()
    lg = lam.cpu().numpy()
    for r in range(6):
        assert np.abs(lg[r] - lam_o[r]).max() <= 1e-10 * np.abs(lam_o[r]).max()
