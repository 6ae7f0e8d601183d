"""The box map's kernel at the edges of its LDS windows (2048 entries of a
workgroup's 256 rows), of its batches of eight entries and of its groups of four
fields, against the oracle's box overlaps."""
import numpy as np
import pytest

import workload as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ns,nr", [((4, 4, 4), (1, 1, 1)), ((20, 20, 20), (2, 1, 1)), ((9, 9, 4), (9, 9, 4)),
                                   ((11, 13, 7), (5, 6, 3)), ((3, 2, 2), (19, 10, 7)), ((30, 30, 10), (16, 17, 1))])
@pytest.mark.parametrize("fields", [1, 2, 3, 4, 5, 8, 11])
@pytest.mark.parametrize("fp64", [False, True])
def test_windows(orc, ns, nr, fields, fp64):
    import torch

    import paper_1807_11834_amd as cpl
    box = (1.0, 1.0, 2.0)
    s, r = W.box_grid(box, ns), W.box_grid(box, nr)
    dt = np.float64 if fp64 else np.float32
    src = np.random.default_rng(fields).normal(size=(fields, s.shape[0])).astype(dt)
    m = cpl.BoxMap(s, r, precision=cpl.COUPLE_FP64 if fp64 else cpl.COUPLE_FP32_WIDE)
    got = m.apply(torch.from_numpy(src).to("cuda")).cpu().numpy().astype(np.float64)
    _, longest = m.info()
    m.close()
    # FP32: the weights and the result rounded once each, sums in FP64; FP64: a
    # rounding per term
    eps = (longest + 4) * 2.0 ** -53 if fp64 else 2.1 * 2.0 ** -24
    for k in range(fields):
        ref, mag = orc.box_remap(src[k], s, r), orc.box_remap(np.abs(src[k]), s, r)
        assert (np.abs(got[k] - ref) <= eps * mag).all()
