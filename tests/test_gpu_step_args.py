"""The one-pass argument check of a step accepts what the general one accepts with the
same addresses, and leaves everything else to it."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _args(cpl, semi, vof, given, prec, n=5):
    cfg = cpl.Config(nb=(3, 2, 4), ratio=2, max_particles=10, semi_implicit=semi, vof=vof, precision=prec,
                     vel_source=cpl.COUPLE_VEL_GIVEN if given else cpl.COUPLE_VEL_FINE)
    z = lambda *s: torch.rand(*s, dtype=cfg.dtype, device="cuda")   # noqa: E731
    inp = {"n": n, "step": 3, "pos": z(n, 3), "vel": z(n, 3), "diam": z(n), "fine_u": z(cfg.n_fine),
           "fine_v": z(cfg.n_fine), "fine_w": z(cfg.n_fine), "fine_p": z(cfg.n_fine),
           "uf_given": z(n, 3) if given else None, "fine_alpha": z(cfg.n_fine) if vof else None}
    return cfg, inp, cpl.alloc_outputs(cfg, n, uf=True)


@pytest.mark.parametrize("semi,vof,given", [(0, 0, 0), (1, 0, 0), (0, 1, 0), (1, 1, 1)])
@pytest.mark.parametrize("fp64", [False, True])
def test_same_addresses(semi, vof, given, fp64):
    import paper_1807_11834_amd as cpl
    cfg, i, o = _args(cpl, semi, vof, given, cpl.COUPLE_FP64 if fp64 else cpl.COUPLE_FP32_WIDE)
    fi, fo = cpl._fast_args(cfg, i, o)
    cpl.validate_step(cfg, i, o)
    assert (fi.n, fi.step) == (5, 3)
    for s, src in ((fi, i), (fo, o)):
        for k, _ in s._fields_:
            if k not in ("n", "step"):
                assert getattr(s, k) == (None if src.get(k) is None else src[k].data_ptr()), k


@pytest.mark.parametrize("bad", ["dtype", "size", "strided", "offset", "cpu", "missing", "type", "capacity", "n", "alpha"])
def test_left_to_the_general_check(bad):
    import paper_1807_11834_amd as cpl
    cfg, i, o = _args(cpl, 0, 1 if bad == "alpha" else 0, 0, cpl.COUPLE_FP32_WIDE)
    if bad == "dtype":
        o["perm"] = o["perm"].long()
    elif bad == "size":
        o["start"] = o["start"][:-1]
    elif bad == "strided":
        i["vel"] = torch.rand(3, 5, device="cuda").t()
    elif bad == "offset":
        i["diam"] = torch.rand(6, device="cuda")[1:]
    elif bad == "cpu":
        o["diag"] = o["diag"].cpu()
    elif bad == "missing":
        o["bulk_G"] = None
    elif bad == "type":
        i["vel"] = [0.0] * 15
    elif bad == "capacity":
        cfg.max_particles = 4
    elif bad == "n":
        i["n"] = 5.0
    else:
        i["fine_alpha"] = None
    assert cpl._fast_args(cfg, i, o) is None
    with pytest.raises(ValueError):
        cpl.validate_step(cfg, i, o)


def test_no_particles_and_subclasses_still_step():
    import paper_1807_11834_amd as cpl
    cfg, i, o = _args(cpl, 0, 0, 0, cpl.COUPLE_FP32_WIDE)
    i["pos"] = torch.nn.Parameter(i["pos"], requires_grad=False)
    assert cpl._fast_args(cfg, i, o) is None
    h = cpl.couple_init(cfg)
    cpl.couple_step(h, i, o)
    cpl.couple_step(h, {**i, "n": 0, "pos": None, "vel": None, "diam": None}, {**cpl.alloc_outputs(cfg, 0)})
    torch.cuda.synchronize()
    cpl.couple_free(h)
