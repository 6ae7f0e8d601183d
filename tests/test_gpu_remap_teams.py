"""The row kernel of the rectilinear transfer where a workgroup's waves share a
receiver row: at both edges of its rules (receiver rows over all fields, bytes of a
sender row), with 16-byte loads or not, and sender rows shorter than the lanes."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sn,dn,fields", [
    ((512, 40, 40), (40, 32, 31), 1),     # 992 receiver rows, teams; half of the lanes load
    ((512, 40, 40), (40, 32, 32), 1),     # 1024: a wave each
    ((508, 40, 40), (40, 8, 16), 8),      # 1024 over eight fields
    ((37, 30, 20), (30, 9, 7), 2),        # short rows, teams
    ((1792, 6, 5), (1000, 3, 2), 3),      # 7 KB in FP32
    ((1796, 42, 40), (30, 34, 32), 1),    # just longer, many rows
    ((896, 42, 40), (30, 34, 32), 1), ((898, 42, 40), (30, 34, 32), 1),   # the same in FP64
    ((3001, 9, 9), (700, 4, 4), 1),       # 81 terms a row from long rows, one value per load
])
@pytest.mark.parametrize("precision", ["wide", "naive", "fp64"])
def test_teams(orc, sn, dn, fields, precision):
    import torch

    import paper_1807_11834_amd as cpl
    prec = {"wide": cpl.COUPLE_FP32_WIDE, "naive": cpl.COUPLE_FP32_NAIVE, "fp64": cpl.COUPLE_FP64}[precision]
    rng = np.random.default_rng(sn[0] + fields)

    def nodes(n):
        e = np.cumsum(rng.uniform(0.5, 1.5, n + 1))
        return (e - e[0]) / (e[-1] - e[0])
    s, d = [nodes(n) for n in sn], [nodes(n) for n in dn]
    dt = np.float64 if precision == "fp64" else np.float32
    src = rng.normal(size=(fields, sn[2], sn[1], sn[0])).astype(dt)
    m = cpl.Remap(s, d, precision=prec)
    got = m.apply(torch.from_numpy(src).to("cuda")).cpu().numpy().astype(np.float64)
    m.close()
    # FP32: the product of three rounded weights, a compensated sum along (z, y),
    # one along x, two stores; plain sums: a rounding per term
    terms = float(np.prod([3.0 * sn[a] / dn[a] + 2 for a in range(3)]))
    eps = {"fp64": terms * 2.0 ** -52, "naive": (terms + 12) * 2.0 ** -24, "wide": 12 * 2.0 ** -24}[precision]
    for f in range(fields):
        ref, mag = orc.remap(src[f], s, d), orc.remap(np.abs(src[f]), s, d)
        assert (np.abs(got[f] - ref) <= eps * mag).all()
