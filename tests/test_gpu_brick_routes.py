"""The fine lookup at ratios 1 and 2 on both sides of its split (512 bricks of 8 x 4
x 2 bulk cells or fewer, and more; bricks cut off at the upper faces; few and many
particles per brick): the velocity at each particle, the restricted velocity and,
through the drag factor, the void fraction, against 64 bits."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

RHO, MU = 1000.0, 1.0e-3


def trilinear(f, pos, h):
    """Value of the cell-centred field f [z, y, x] at pos, nodes clamped at the walls."""
    n = f.shape[::-1]
    g = pos / h - 0.5
    lo = np.floor(g).astype(np.int64)
    t = g - lo
    out = 0.0
    for c in range(8):
        k = [(c >> a) & 1 for a in range(3)]
        i = [np.clip(lo[:, a] + k[a], 0, n[a] - 1) for a in range(3)]
        w = np.prod([t[:, a] if k[a] else 1.0 - t[:, a] for a in range(3)], axis=0)
        out = out + w * f[i[2], i[1], i[0]]
    return out


@pytest.mark.parametrize("nb", [(64, 32, 16), (65, 32, 16), (3, 60, 70)])
@pytest.mark.parametrize("ratio", [1, 2])
@pytest.mark.parametrize("n,cic", [(500, True), (60_000, False), (60_000, True)])
@pytest.mark.parametrize("precision", ["wide", "kahan", "fp64"])
def test_lookup(nb, ratio, n, cic, precision):
    import torch

    import paper_1807_11834_amd as cpl
    prec = {"wide": cpl.COUPLE_FP32_WIDE, "kahan": cpl.COUPLE_FP32_KAHAN, "fp64": cpl.COUPLE_FP64}[precision]
    dt = np.float64 if precision == "fp64" else np.float32
    u = 2.0 ** -53 if precision == "fp64" else 2.0 ** -24
    h = 1.0 / 64
    box = tuple(c * h for c in nb)
    nf = [c * ratio for c in nb]
    rng = np.random.default_rng(sum(nb) + n)
    pos = (rng.random((n, 3)) * box).astype(dt)
    vel = (0.1 * rng.normal(size=(n, 3))).astype(dt)
    # spheres of a mean solid fraction of 0.02 or less and no more than half a cell's width
    diam = np.full(n, min(0.5, (0.02 * np.prod(nb) / n * 6.0 / np.pi) ** (1.0 / 3.0)) * h).astype(dt)
    fine = rng.normal(size=(4, nf[2], nf[1], nf[0])).astype(dt)
    cfg = cpl.Config(box=box, nb=nb, ratio=ratio, rho_f=RHO, mu_f=MU, eps_min=0.1,
                     deposit=cpl.COUPLE_CIC if cic else cpl.COUPLE_NGP, precision=prec, max_particles=n)
    put = lambda a: torch.from_numpy(a).to("cuda:0")
    print(f"case {nb} r{ratio} n{n} cic={cic} {precision}", flush=True)
    c = cpl.Coupler(cfg)
    out = c.step(put(pos), put(vel), put(diam), [put(f) for f in fine], uf=True)
    g = {k: out[k].cpu().numpy().astype(np.float64) for k in ("uf", "bulk_U", "bulk_phi", "beta", "cell")}
    c.close()
    p64, f64 = pos.astype(np.float64), fine.astype(np.float64)
    # a position in node units is off by a rounded scale and one rounding, on each axis,
    # which moves the value by at most that times the spread of the nodes; then the
    # roundings of three interpolations
    spread = f64[:3].max() - f64[:3].min()
    tol = (2.0 * sum(nf) * spread + 16.0 * np.abs(f64[:3]).max()) * u
    ref = np.stack([trilinear(f64[k], p64, h / ratio) for k in range(3)], 1)
    assert np.abs(g["uf"] - ref).max() <= tol
    # averages of r^3 children: a rounding per child at most
    kids = f64[:3].reshape(3, nb[2], ratio, nb[1], ratio, nb[0], ratio)
    assert (np.abs(g["bulk_U"].reshape(3, nb[2], nb[1], nb[0]) - kids.mean((2, 4, 6)))
            <= ratio ** 3 * u * np.abs(kids).mean((2, 4, 6)) + u).all()
    # void fraction: from the library's own phi, in the drag factor
    phi = g["bulk_phi"].reshape(nb[2], nb[1], nb[0])
    eps = 1.0 - (trilinear(phi, p64, h) if cic else phi.ravel()[g["cell"].astype(np.int64)])
    assert eps.min() > 0.1
    mag = np.sqrt(((g["uf"] - vel.astype(np.float64)) ** 2).sum(1))
    d = diam.astype(np.float64)
    re = RHO * eps * d * mag / MU
    chi = 3.7 - 0.65 * np.exp(-0.5 * (1.5 - np.log10(re)) ** 2)
    beta = (0.5 * RHO * np.pi / 4.0 * d * d * eps ** (2.0 - chi)
            * (0.63 * np.sqrt(mag) + 4.8 * np.sqrt(MU / (RHO * eps * d))) ** 2)
    # eps off by the stencil's error; beta ~ eps^(2 - chi) / eps at most; 64 roundings of
    # the formula (its functions among them)
    deps = (2.0 * sum(nb) * phi.max() + 16.0) * u
    assert (np.abs(g["beta"] / beta - 1.0) <= 3.0 * deps / eps.min() + 64.0 * u).all()
