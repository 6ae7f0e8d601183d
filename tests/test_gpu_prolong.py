"""The prolongation at the edges of its tile widths (128 x 2 to 16 x 16 bulk cells)
and with more work items than diagnostic partials, against the oracle's
prolongation of the step's own bulk fields."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

# (nb, ratio, particles): widths 16, 32, 64, 128 with and without remainders; one-cell
# axes; a flat grid of many items, whose partials are fewer
GRIDS = [((1, 1, 1), 4, 5), ((16, 17, 2), 2, 300), ((17, 5, 3), 4, 300), ((33, 9, 2), 4, 500), ((64, 4, 3), 4, 500),
         ((65, 5, 2), 2, 500), ((128, 2, 3), 4, 500), ((129, 3, 1), 1, 500), ((256, 3, 2), 4, 900),
         ((3, 40, 700), 4, 64), ((3, 3, 1300), 4, 64)]


@pytest.mark.parametrize("nb,ratio,n", GRIDS)
@pytest.mark.parametrize("precision", ["wide", "fp64"])
def test_tile_widths(orc, nb, ratio, n, precision):
    import paper_1807_11834_amd as cpl
    f64 = precision == "fp64"
    dt = torch.float64 if f64 else torch.float32
    g = torch.Generator(device="cuda")
    g.manual_seed(sum(nb))
    box = tuple(0.25 * m for m in nb)
    kw = dict(generator=g, device="cuda", dtype=dt)
    pos = torch.rand((n, 3), **kw) * torch.tensor(box, dtype=dt, device="cuda")
    vel, diam = torch.randn((n, 3), **kw), 0.05 + 0.05 * torch.rand((n,), **kw)
    cfg = cpl.Config(box=box, nb=nb, ratio=ratio, precision=cpl.COUPLE_FP64 if f64 else cpl.COUPLE_FP32_WIDE,
                     max_particles=n, semi_implicit=1)
    fine = [torch.randn(cfg.nf[::-1], **kw) for _ in range(4)]
    c = cpl.Coupler(cfg)
    out = c.step(pos, vel, diam, fine)
    torch.cuda.synchronize()
    d = cpl.diag_dict(out["diag"])
    h = lambda t: t.cpu().numpy().astype(np.float64)
    bulk = [1.0 - h(out["bulk_phi"])] + list(h(out["bulk_F"])) + [h(out["bulk_K"])] + list(h(out["bulk_KU"]))
    got = [h(out["fine_eps"])] + list(h(out["fine_F"])) + [h(out["fine_K"])] + list(h(out["fine_KU"]))
    sums = [d["E_f"], *d["S_f"], d["K_f"], *d["KU_f"]]
    # a child is a sum of weighted bulk values, |weights| summing to at most 4 (the
    # trilinear part and the defect), through at most 24 roundings
    eps = (2.0 ** -53 if f64 else 2.0 ** -24) * 24 * 4
    vf = np.prod(box) / got[0].size
    for B, f, s in zip(bulk, got, sums):
        ref = orc.prolong(B, nb, ratio)
        assert np.abs(f.ravel() - ref).max() <= eps * max(1.0, np.abs(B).max())
        # the FP64 sum over the children as they were stored
        assert abs(s - f.sum() * vf) <= 1e-12 * np.abs(f).sum() * vf
    c.close()


@pytest.mark.parametrize("nb", [(4, 4, 4), (5, 13, 1), (7, 9, 10), (40, 30, 20)])
@pytest.mark.parametrize("n", [0, 1, 700, 6000])
def test_ngp_workgroups(nb, n):
    """Containing-cell sums at the edges of a workgroup's 64 cells and of its
    chunks of particles, FP64: against torch's sums per cell."""
    import paper_1807_11834_amd as cpl
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    kw = dict(generator=g, device="cuda", dtype=torch.float64)
    pos, vel, diam = torch.rand((n, 3), **kw), torch.randn((n, 3), **kw), 0.01 + 0.01 * torch.rand((n,), **kw)
    pos[: n // 2] *= 0.2                      # some cells with many particles, many with none
    cfg = cpl.Config(nb=nb, ratio=1, deposit=cpl.COUPLE_NGP, precision=cpl.COUPLE_FP64, max_particles=n)
    fine = [torch.randn(cfg.nf[::-1], **kw) for _ in range(4)]
    c = cpl.Coupler(cfg)
    out = c.step(pos, vel, diam, fine)
    nc = cfg.n_bulk
    ref = torch.zeros((4, nc), dtype=torch.float64, device="cuda")
    src = torch.cat([np.pi / 6 * diam[None] ** 3, -out["drag"].T])
    ref.index_add_(1, out["cell"].long(), src)
    mag = torch.zeros_like(ref).index_add_(1, out["cell"].long(), src.abs())
    got = torch.cat([out["bulk_phi"].reshape(1, -1), out["bulk_F"].reshape(3, -1)]) / nc
    # at most n + 4 roundings of terms whose magnitudes sum to mag
    assert bool(((got - ref).abs() <= (n + 4) * 2.0 ** -53 * mag).all())
    d = out["diag"]
    assert torch.allclose(torch.cat([d[1:2], d[5:8]]), ref.sum(1), rtol=1e-10, atol=1e-12 * float(mag.sum() + 1e-300))
    assert float(d[14]) == float(out["bulk_phi"].max())
    c.close()
