"""The deposit's work list where a tile holds more items than its thread writes (32): one tile of a
grid, a tile at that count and one past it, and more such tiles (512) than the workgroup takes
together (128).  The charge is summed as integers, so it does not depend on the items: the bits of
the largest items' list, whose tiles hold a few."""
import pytest
import torch

import paper_2208_02382_amd as pic
import workloads

pytestmark = pytest.mark.gpu


def _rho(X, nodes, tile, chunk):
    cfg = workloads.SMALL
    b = pic.Beam(X.shape[1], cfg.qm_qeeV, cfg.charge_C, cfg.kin_energy_MeV, cfg.mass_MeV, 1, nodes,
                 tuning={"tile": tile, "chunk": chunk})
    b.X.copy_(X)
    rho = b.deposit().clone()
    assert b.check() == pic.PIC_OK
    b.close()
    return rho


@pytest.mark.parametrize("n,nodes,tile", [(32 * 256, (4, 4, 4), (4, 4, 4)),
                                          (32 * 256 + 1, (4, 4, 4), (4, 4, 4)),
                                          (1_300_001, (8, 8, 8), (4, 4, 8)),
                                          (9_000_000, (16, 16, 16), (2, 2, 2))])
def test_every_item_is_in_the_list(n, nodes, tile):
    g = torch.Generator(device="cuda").manual_seed(n)
    X = torch.rand((6, n), generator=g, dtype=torch.float64, device="cuda") - 0.5
    assert torch.equal(_rho(X, nodes, tile, 256), _rho(X, nodes, tile, 1 << 20))


@pytest.mark.parametrize("n,nodes", [(786_431, (4, 4, 4)), (786_432, (4, 4, 4)),
                                     (884_735, (12, 12, 12)), (884_736, (12, 12, 12)),
                                     (3_200_000, (8, 12, 16))])
def test_default_items_on_grids_of_few_tiles(n, nodes):
    """Around the counts where the default items grow from 512 on 1 and 27 tiles, and on 24 tiles."""
    g = torch.Generator(device="cuda").manual_seed(n)
    X = 1e-3 * torch.randn((6, n), generator=g, dtype=torch.float64, device="cuda")
    assert torch.equal(_rho(X, nodes, (0, 0, 0), 0), _rho(X, nodes, (0, 0, 0), 8192))
