"""The FP64 diagnostics of a step are the same bits whatever the capacity of the
scratch it runs in: a handle for exactly its particles, one for many more, and the
static scratch (also where that is nearly full and holds the fewest sort tiles).
Grids whose kernels loop over their work: containing-cell sums over more groups than
other kernels have workgroups, prolongation tiles that pad a thin layer."""
import pytest

import workload as W
from parity_util import cfg_for, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nb,ratio,n,deposit,precision", [
    ((64, 64, 64), 1, 2000, "ngp", "fp32"), ((64, 64, 64), 1, 2000, "ngp", "fp64"),
    ((100, 1, 1500), 1, 2000, "cic", "fp32"), ((20, 20, 20), 2, 1_340_000, "cic", "fp32"),
    ((20, 20, 20), 2, 1_340_000, "ngp", "fp32")])
def test_capacity(nb, ratio, n, deposit, precision):
    import torch

    import paper_1807_11834_amd as cpl
    box = tuple(0.01 * c for c in nb)
    w = W.small_workload(nb=nb, ratio=ratio, box=box, n=n, seed=905, precision=precision, deposit=deposit)
    pos, d, vel = W.particles(w)
    n = pos.shape[0]
    cfg = cfg_for(cpl, w, n)
    put = lambda a: to_dev(a, torch, "cuda:0", cfg.dtype)
    fine = [put(f) for f in W.fine_fields(w)]
    inp = {"n": n, "pos": put(pos), "vel": put(vel), "diam": put(d), "fine_u": fine[0], "fine_v": fine[1],
           "fine_w": fine[2], "fine_p": fine[3]}
    outs = []
    for capacity in (n, n + 1_000_000, None):
        out = cpl.alloc_outputs(cfg, n, device="cuda:0")
        if capacity is None:
            cpl.couple_step_noalloc(cfg, inp, out)
        else:
            h = cpl.couple_init(cpl.Config(**{**cfg.__dict__, "max_particles": capacity}))
            cpl.couple_step(h, inp, out)
            torch.cuda.synchronize()
            cpl.couple_free(h)
        outs.append(out)
    torch.cuda.synchronize()
    for o in outs[1:]:
        for k, t in outs[0].items():
            assert t is None or torch.equal(t, o[k]), k
