"""The counting sort of few particles in few cells and its limits (8192 cells, 65,535
particles, tiles of 1024): cell, perm, count and start against torch's stable sort
(whole numbers, equal), and the static-scratch step against the allocating one."""
import pytest
import torch

pytestmark = pytest.mark.gpu

GRIDS = [(1, 1, 1), (7, 1, 1), (3, 3, 1), (7, 5, 9), (16, 16, 8), (23, 89, 1), (16, 16, 32), (8193, 1, 1)]


def _inputs(n, nb, clustered, dev="cuda"):
    g = torch.Generator(device=dev)
    g.manual_seed(n + nb[0])
    pos = torch.rand((n, 3), generator=g, device=dev)
    if clustered:      # nine tenths in one cell, and the rest leaving long runs of cells empty
        pos[: 9 * n // 10] = torch.tensor([0.999, 0.999, 0.999], device=dev)
        pos = pos[torch.randperm(n, generator=g, device=dev)].contiguous()
    return pos, torch.zeros_like(pos), torch.full((n,), 1e-3, device=dev), \
        [torch.zeros(nb[::-1], device=dev) for _ in range(4)]


def _check(out, pos, nb):
    t = torch.tensor(nb, device=pos.device)
    c = torch.minimum((pos * t).floor().long().clamp(min=0), t - 1)
    cell = c[:, 0] + nb[0] * (c[:, 1] + nb[1] * c[:, 2])
    count = torch.bincount(cell, minlength=nb[0] * nb[1] * nb[2])
    assert torch.equal(out["cell"].long(), cell)
    assert torch.equal(out["perm"].long(), torch.argsort(cell, stable=True))
    assert torch.equal(out["count"].reshape(-1).long(), count)
    assert torch.equal(out["start"].long(), torch.cat([count.new_zeros(1), count.cumsum(0)]))


@pytest.mark.parametrize("nb", GRIDS)
@pytest.mark.parametrize("n", [1, 65, 1024, 1025, 8 * 1024 + 1, 65_535, 65_536])
@pytest.mark.parametrize("clustered", [False, True])
def test_edges(nb, n, clustered):
    import paper_1807_11834_amd as cpl
    pos, vel, diam, fine = _inputs(n, nb, clustered)
    cfg = cpl.Config(nb=nb, ratio=1, deposit=cpl.COUPLE_NGP, max_particles=n)
    c = cpl.Coupler(cfg)
    for _ in range(2):      # the second step finds the first's histograms in its scratch
        _check(c.step(pos, vel, diam, fine), pos, nb)
    c.close()
    out = cpl.alloc_outputs(cfg, n)
    cpl.couple_step_noalloc(cfg, {"n": n, "pos": pos, "vel": vel, "diam": diam, "fine_u": fine[0], "fine_v": fine[1],
                                  "fine_w": fine[2], "fine_p": fine[3]}, out)
    _check(out, pos, nb)
