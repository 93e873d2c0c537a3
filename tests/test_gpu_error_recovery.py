"""A beam that ended a call in a device error and is initialised again is as good as a new one: its
next calls give the bits of a fresh beam's.  At the sizes where the return to the caller's order
counts the particles' labels in the histogram that the ranking uses (above 2^20 particles, and in
every batch)."""
import pytest
import torch

import paper_2208_02382_amd as pic
import workloads

pytestmark = pytest.mark.gpu

FODO = ((1.0, 0.5), (-1.0, 0.5))


def _beam(n, nodes):
    cfg = workloads.SMALL
    b = pic.Beam(n, cfg.qm_qeeV, cfg.charge_C, cfg.kin_energy_MeV, cfg.mass_MeV, 1, nodes)
    b.init(cfg.sigma_matrix, seed=3)
    return b


def _spoil_and_restart(b, track):
    b.X[2, b.X.shape[1] // 2] = float("nan")
    track()
    assert b.check() == pic.PIC_EDOMAIN
    b.init(workloads.SMALL.sigma_matrix, seed=3)
    assert b.check() == pic.PIC_OK


@pytest.mark.parametrize("n", [(1 << 20) + 1, 1_500_000])
@pytest.mark.parametrize("steps", [1, 3])
def test_tracking_and_deposit_after_an_error(n, steps):
    used, fresh = _beam(n, (32, 32, 32)), _beam(n, (32, 32, 32))
    _spoil_and_restart(used, lambda: used.track(FODO, steps))
    assert torch.equal(used.deposit(), fresh.deposit())
    for b in (used, fresh):
        b.track(FODO, 2)
        assert b.check() == pic.PIC_OK
    assert torch.equal(used.X, fresh.X)
    used.close()
    fresh.close()


def test_a_batch_after_one_beams_error():
    ns = (1000, 70_001, 5000)
    used, fresh = ([_beam(n, (16, 16, 16)) for n in ns] for _ in range(2))
    bu, bf = (pic.Batch(beams, [FODO] * len(ns)) for beams in (used, fresh))
    _spoil_and_restart(used[1], lambda: bu.track(2))
    for b in (used[0], used[2]):
        assert b.check() == pic.PIC_OK
        b.init(workloads.SMALL.sigma_matrix, seed=3)
    bu.track(3)
    bf.track(3)
    for u, f in zip(used, fresh):
        assert u.check() == pic.PIC_OK and f.check() == pic.PIC_OK
        assert torch.equal(u.X, f.X)
    # a beam's own calls take over from the batch's
    _spoil_and_restart(used[1], lambda: bu.track(2))
    fresh[1].init(workloads.SMALL.sigma_matrix, seed=3)
    assert torch.equal(used[1].deposit(), fresh[1].deposit())
    bu.close()
    bf.close()
    for b in used + fresh:
        b.close()
