"""The slice-step diagnostics against float64 moments of the state they describe, at a few particles,
around a wavefront, and on both sides of the particle counts where the workgroup count changes; a
second run on the same beam finds the accumulators of the first.

Tolerance: the sums have at most n / (512 * 256) + 200 terms in a row, so each carries under 460
rounding errors of 1.1e-16 relative to the sum of its terms' magnitudes, 5e-14; the shift (grid
centre, then the previous step's mean) lies within about an rms of the mean for these beams, which
multiplies the centred products' terms by at most 4: 2e-13, and 1e-12 is asked of each entry
relative to its rms product."""
import pytest
import torch

import paper_2208_02382_amd as pic
import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [5, 63, 4097, 1 << 21, (1 << 21) + 1, 1 << 25, (1 << 25) + 1])
def test_diagnostics_equal_the_moments_of_the_state(n):
    cfg = workloads.MEDIUM
    b = pic.Beam(n, cfg.qm_qeeV, cfg.charge_C, cfg.kin_energy_MeV, cfg.mass_MeV, 1, (32, 32, 32))
    b.init(cfg.sigma_matrix, seed=11)
    sig = torch.tensor(cfg.sigma_matrix, dtype=torch.float64).cuda()
    floor = sig.diagonal().sqrt()
    iu = torch.triu_indices(6, 6)
    for _ in range(2):
        d = b.track(cfg.lattice, 3, diagnostics=True)[-1]
        mean = b.X.mean(dim=1)
        dx = b.X - mean[:, None]
        cov = dx @ dx.T / n
        rms = torch.maximum(cov.diagonal().sqrt(), floor)
        assert ((d[:6] - mean).abs() / rms).max().item() < 1e-12
        prod = rms[iu[0]] * rms[iu[1]]
        assert ((d[6:] - cov[iu[0], iu[1]]).abs() / prod).max().item() < 1e-12
    assert b.check() == pic.PIC_OK
    b.close()
