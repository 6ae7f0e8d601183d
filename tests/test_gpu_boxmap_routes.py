"""The box map's three ways through a workgroup's entries: windows in LDS, long rows
and rows of one or two entries from memory, and a grid whose workgroups differ,
against the oracle's box overlaps."""
import numpy as np
import pytest

import workload as W

pytestmark = pytest.mark.gpu

BOX = (1.0, 1.0, 2.0)


@pytest.mark.parametrize("ns,nr", [
    ((26, 26, 26), (8, 8, 4)),      # 5 x 5 x 8 entries a row: long rows, a whole workgroup
    ((24, 24, 24), (13, 11, 3)),    # some 70 a row, workgroups that end inside a row's run
    ((24, 24, 24), (11, 9, 9)),     # some 40: five windows, FP64 through LDS and FP32 not
    ((5, 4, 3), (20, 16, 15)),      # one entry a row
    ((5, 4, 3), (22, 17, 13)),      # one to eight, about two
    ((24, 24, 24), (2, 2, 1)),      # four receivers: 3456 entries each
    ((9, 9, 9), (3, 3, 1)),         # nine of some 81 entries
    ((4, 4, 4), (2, 2, 1)),         # four of sixteen
])
@pytest.mark.parametrize("refined", [False, True])
@pytest.mark.parametrize("fields", [1, 4, 7])
@pytest.mark.parametrize("precision", ["wide", "kahan", "fp64"])
def test_routes(orc, ns, nr, refined, fields, precision):
    import torch

    import paper_1807_11834_amd as cpl
    prec = {"wide": cpl.COUPLE_FP32_WIDE, "kahan": cpl.COUPLE_FP32_KAHAN, "fp64": cpl.COUPLE_FP64}[precision]
    s, r = W.box_grid(BOX, ns), W.box_grid(BOX, nr)
    if refined:
        s = W.refined_box_grid(BOX, ns, (-1.0, 2.0, -1.0, 2.0, -1.0, 0.5))
        s = s[0] if isinstance(s, tuple) else s
    dt = np.float64 if precision == "fp64" else np.float32
    src = np.random.default_rng(fields).normal(size=(fields, s.shape[0])).astype(dt)
    m = cpl.BoxMap(s, r, precision=prec)
    got = m.apply(torch.from_numpy(src).to("cuda")).cpu().numpy().astype(np.float64)
    _, longest = m.info()
    m.close()
    # FP32: the weights and the result rounded once each, sums in FP64 or
    # compensated (a rounding of the last sum and its residue more); FP64: a rounding
    # per term
    eps = {"fp64": (longest + 4) * 2.0 ** -53, "wide": 2.1 * 2.0 ** -24, "kahan": 4.1 * 2.0 ** -24}[precision]
    for k in range(fields):
        ref, mag = orc.box_remap(src[k], s, r), orc.box_remap(np.abs(src[k]), s, r)
        assert (np.abs(got[k] - ref) <= eps * mag).all()
