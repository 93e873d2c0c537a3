"""The return to the caller's order at the sizes where its form changes: the largest direct
return, the smallest bucketed one, and buckets of 8192 and 16384 particles (the last of them
short).  Moving particles rounds nothing, so the result equals the binned order's, put back by
its labels, bit for bit."""
import pytest
import torch

import paper_2208_02382_amd as pic
import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1 << 20, (1 << 20) + 1, (1 << 24) + 1, (1 << 25) + 4097])
def test_return_to_the_callers_order(n):
    cfg = workloads.MEDIUM
    out = []
    for binned in (False, True):
        b = pic.Beam(n, cfg.qm_qeeV, cfg.charge_C, cfg.kin_energy_MeV, cfg.mass_MeV, 1,
                     (16, 16, 16))
        b.init(cfg.sigma_matrix, seed=7)
        if binned:
            ids = torch.arange(n, dtype=torch.int32, device="cuda")
            b.track(cfg.lattice, 2, binned=True, ids=ids)
            X = torch.empty_like(b.X)
            X[:, ids.long()] = b.X
            out.append(X)
        else:
            b.track(cfg.lattice, 2)
            out.append(b.X.clone())
        assert b.check() == pic.PIC_OK
        b.close()
    assert torch.equal(out[0], out[1])
