"""The prolongation of ratio 4 on grids of many tiles, whose width follows from the
type and the length of x (16, 64 or 128 cells, with and without remainders), against
the oracle's prolongation of the step's own bulk fields."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nb", [(8, 30, 65), (9, 30, 65), (16, 30, 64), (16, 30, 65), (17, 30, 65), (72, 9, 90), (72, 9, 80), (128, 8, 128),
                                (105, 7, 130), (129, 5, 90)])
@pytest.mark.parametrize("precision", ["wide", "fp64"])
def test_widths(orc, nb, precision):
    import paper_1807_11834_amd as cpl
    f64 = precision == "fp64"
    dt = torch.float64 if f64 else torch.float32
    n = 500
    g = torch.Generator(device="cuda")
    g.manual_seed(sum(nb))
    box = tuple(0.25 * m for m in nb)
    kw = dict(generator=g, device="cuda", dtype=dt)
    pos = torch.rand((n, 3), **kw) * torch.tensor(box, dtype=dt, device="cuda")
    vel, diam = torch.randn((n, 3), **kw), 0.05 + 0.05 * torch.rand((n,), **kw)
    cfg = cpl.Config(box=box, nb=nb, ratio=4, precision=cpl.COUPLE_FP64 if f64 else cpl.COUPLE_FP32_WIDE, max_particles=n)
    c = cpl.Coupler(cfg)
    out = c.step(pos, vel, diam, [torch.randn(cfg.nf[::-1], **kw) for _ in range(4)])
    torch.cuda.synchronize()
    d = cpl.diag_dict(out["diag"])
    h = lambda t: t.cpu().numpy().astype(np.float64)
    bulk = [1.0 - h(out["bulk_phi"])] + list(h(out["bulk_F"]))
    got = [h(out["fine_eps"])] + list(h(out["fine_F"]))
    c.close()
    # a child is a sum of weighted bulk values, |weights| summing to at most 4 (the
    # trilinear part and the defect), through at most 24 roundings
    eps = (2.0 ** -53 if f64 else 2.0 ** -24) * 24 * 4
    vf = np.prod(box) / got[0].size
    for B, f, s in zip(bulk, got, [d["E_f"], *d["S_f"]]):
        assert np.abs(f.ravel() - orc.prolong(B, nb, 4)).max() <= eps * max(1.0, np.abs(B).max())
        assert abs(s - f.sum() * vf) <= f.size * 2.0 ** -53 * np.abs(f).sum() * vf
