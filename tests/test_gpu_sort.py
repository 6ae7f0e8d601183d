"""The binning and the radix sort at the edges of their tile sizes: cell, perm, count
and start against torch's stable sort (whole numbers, equal)."""
import pytest
import torch

pytestmark = pytest.mark.gpu

NB = (7, 5, 9)
TILE4, WANTED = 1024, 1024      # keys of the smallest tile; tiles above which tiles grow


def _inputs(n, dev="cuda"):
    g = torch.Generator(device=dev)
    g.manual_seed(n)
    pos = torch.rand((n, 3), generator=g, device=dev)
    return pos, torch.zeros_like(pos), torch.full((n,), 1e-3, device=dev), \
        [torch.zeros(NB[::-1], device=dev) for _ in range(4)]


def _check(out, pos, n):
    nb = torch.tensor(NB, device=pos.device)
    c = (pos * nb).floor().long().clamp(min=0)
    c = torch.minimum(c, nb - 1)
    cell = c[:, 0] + NB[0] * (c[:, 1] + NB[1] * c[:, 2])
    count = torch.bincount(cell, minlength=NB[0] * NB[1] * NB[2])
    assert torch.equal(out["cell"].long(), cell)
    assert torch.equal(out["perm"].long(), torch.argsort(cell, stable=True))
    assert torch.equal(out["count"].reshape(-1).long(), count)
    assert torch.equal(out["start"].long(), torch.cat([count.new_zeros(1), count.cumsum(0)]))


@pytest.mark.parametrize("n", [1, 63, 1023, 1024, 1025, 4097, TILE4 * WANTED, TILE4 * WANTED + 1, 2 * TILE4 * WANTED,
                               2 * TILE4 * WANTED + 1])
@pytest.mark.parametrize("spare", [0, 3_000_000])
def test_tile_edges(n, spare):
    import paper_1807_11834_amd as cpl
    pos, vel, diam, fine = _inputs(n)
    c = cpl.Coupler(cpl.Config(nb=NB, ratio=1, deposit=cpl.COUPLE_NGP, max_particles=n + spare))
    _check(c.step(pos, vel, diam, fine), pos, n)
    c.close()


def test_noalloc_at_the_scratch_limit():
    """The largest step the static scratch holds sorts with its largest tiles."""
    import paper_1807_11834_amd as cpl
    cfg = cpl.Config(nb=NB, ratio=1, deposit=cpl.COUPLE_NGP)
    pos, vel, diam, fine = _inputs(1_500_000)

    def step(n):
        out = cpl.alloc_outputs(cfg, n)
        cpl.couple_step_noalloc(cfg, {"n": n, "pos": pos[:n], "vel": vel[:n], "diam": diam[:n], "fine_u": fine[0],
                                      "fine_v": fine[1], "fine_w": fine[2], "fine_p": fine[3]}, out)
        return out
    lo, hi = 1_000_000, pos.shape[0]
    while hi - lo > 1:
        mid = (lo + hi) // 2
        try:
            step(mid)
            lo = mid
        except cpl.CoupleError:
            hi = mid
    # 16 B of keys and values, 32 B of records, 1/4 B of histograms and one FP64
    # partial per 31 slots and 256 particles
    assert lo * (48 + 0.25 + 31 * 8 / 256) > 0.999 * cpl.NOALLOC_SCRATCH_BYTES
    _check(step(lo), pos[:lo], lo)
