"""The reverse sweep of millions of particles, whose deposits read them through their ranking as
records, against the oracle; on both sides of the count whose rows fill the memory-side cache.

A wrong order is an error of order one.  Bar 1e-10: the rounding of sums over 5.6e6 particles (chains
of at most about 2000 terms here, 2e-13, pairwise in the oracle), times 100 for the geometry terms,
whose sums over the particles cancel."""
import numpy as np
import pytest
import torch

import workloads
from oracle import adjoint as oadj
from oracle import pic as opic

pytestmark = pytest.mark.gpu

EDGE = (256 << 20) // 48


@pytest.mark.parametrize("n", [EDGE, EDGE + 1])
def test_reverse_sweep_of_millions_of_particles(n):
    import paper_2208_02382_amd as lib
    cfg = workloads.SMALL
    nodes, w4 = (12, 12, 12), np.array([0.7, -0.4, 1.3, 0.9])
    xi = np.random.default_rng(3).standard_normal((6, n))
    prob = opic.make_problem(n, cfg.qm_qeeV, cfg.charge_C, cfg.kin_energy_MeV, cfg.mass_MeV,
                             nodes, 1)
    X0 = opic.init_from_normals(cfg.sigma_matrix, xi)
    _, dk_o, lam_o, _ = oadj.adjoint(X0, np.array([1.0]), np.array([0.5]), 1, prob, w4)
    b = lib.Beam(n, cfg.qm_qeeV, cfg.charge_C, cfg.kin_energy_MeV, cfg.mass_MeV, 1, nodes)
    b.init_from_normals(cfg.sigma_matrix, torch.from_numpy(xi).cuda())
    _, dk, lam, _ = b.track_adjoint(((1.0, 0.5),), 1, w4, ckpt_every=1)
    b.close()
    assert np.abs(np.array(dk) - dk_o).max() <= 1e-10 * np.abs(dk_o).max()
    lg = lam.cpu().numpy()
    for r in range(6):
        assert np.abs(lg[r] - lam_o[r]).max() <= 1e-10 * np.abs(lam_o[r]).max()
