"""The prolongation at ratio 1 is a copy: the fine fields are the bulk ones bit for bit
(the porosity 1 - phi), over whole tiles, cut-off ones and more of them than
workgroups, and their sums are the FP64 sums of what was stored."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nb", [(1, 1, 1), (129, 3, 5), (100, 2, 700), (3, 40, 90), (64, 64, 8)])
@pytest.mark.parametrize("precision", ["wide", "fp64"])
@pytest.mark.parametrize("semi", [0, 1])
def test_copy(nb, precision, semi):
    import paper_1807_11834_amd as cpl
    f64 = precision == "fp64"
    n = 2000
    g = torch.Generator(device="cuda")
    g.manual_seed(sum(nb))
    box = tuple(0.25 * m for m in nb)
    kw = dict(generator=g, device="cuda", dtype=torch.float64 if f64 else torch.float32)
    pos = torch.rand((n, 3), **kw) * torch.tensor(box, dtype=kw["dtype"], device="cuda")
    vel, diam = torch.randn((n, 3), **kw), 0.05 + 0.05 * torch.rand((n,), **kw)
    cfg = cpl.Config(box=box, nb=nb, ratio=1, precision=cpl.COUPLE_FP64 if f64 else cpl.COUPLE_FP32_WIDE,
                     max_particles=n, semi_implicit=semi)
    c = cpl.Coupler(cfg)
    out = c.step(pos, vel, diam, [torch.randn(cfg.nf[::-1], **kw) for _ in range(4)])
    pairs = [(out["fine_eps"], 1.0 - out["bulk_phi"], "E_f"), (out["fine_F"], out["bulk_F"], "S_f")]
    if semi:
        pairs += [(out["fine_K"], out["bulk_K"], "K_f"), (out["fine_KU"], out["bulk_KU"], "KU_f")]
    d = cpl.diag_dict(out["diag"])
    vf = 0.25 ** 3
    for fine, bulk, name in pairs:
        assert torch.equal(fine.flatten(), bulk.flatten())
        f = fine.double().cpu().numpy().reshape(-1, int(np.prod(nb)))
        # the order of the sum is free
        assert (np.abs(np.atleast_1d(d[name]) - f.sum(1) * vf) <= f.shape[1] * 2.0 ** -53 * np.abs(f).sum(1) * vf).all()
    c.close()
