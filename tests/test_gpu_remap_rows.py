"""The row kernel of the rectilinear transfer at its edges: sender rows that take
16-byte loads or not, one chunk of lanes and more, four rows or one to a
workgroup, more than sixteen (z, y) terms, x factors in LDS or in memory."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sx,dx", [(1, 1), (5, 3), (64, 37), (256, 96), (257, 96), (260, 300), (1024, 500), (3836, 50),
                                   (3844, 1900), (15000, 70)])
@pytest.mark.parametrize("sy,dy,sz,dz", [(4, 2, 5, 2), (11, 2, 9, 1), (3, 3, 2, 2)])
@pytest.mark.parametrize("precision", ["wide", "kahan", "fp64"])
def test_rows(orc, sx, dx, sy, dy, sz, dz, precision):
    import torch

    import paper_1807_11834_amd as cpl
    prec = {"wide": cpl.COUPLE_FP32_WIDE, "kahan": cpl.COUPLE_FP32_KAHAN, "fp64": cpl.COUPLE_FP64}[precision]
    rng = np.random.default_rng(sx + dy)

    def nodes(n):
        e = np.cumsum(rng.uniform(0.5, 1.5, n + 1))
        return (e - e[0]) / (e[-1] - e[0])
    s, d = [nodes(n) for n in (sx, sy, sz)], [nodes(n) for n in (dx, dy, dz)]
    dt = np.float64 if precision == "fp64" else np.float32
    src = rng.normal(size=(2, sz, sy, sx)).astype(dt)
    m = cpl.Remap(s, d, precision=prec)
    got = m.apply(torch.from_numpy(src).to("cuda")).cpu().numpy().astype(np.float64)
    m.close()
    # FP32: the product of three rounded weights, a compensated sum along (z, y),
    # one along x, two stores; FP64: plain sums, a rounding per term
    eps = (sx / dx + 2) * (sy / dy + 2) * (sz / dz + 2) * 2.0 ** -52 if precision == "fp64" else 12 * 2.0 ** -24
    for f in range(2):
        ref, mag = orc.remap(src[f], s, d), orc.remap(np.abs(src[f]), s, d)
        assert (np.abs(got[f].ravel() - np.ravel(ref)) <= eps * np.ravel(mag)).all()
