"""The containing-cell deposition on both sides of its rules for the cells of a group
(256 with at most two particles per cell, then 64 or 16, fewer where a group would
have more than a chunk of 1024 particles), spread or crowded into few cells: solid
fraction, momentum source, K and KU and their sums against 64 bits formed from the
step's own cells and drags, the pressure gradient against the trilinear
deposition's."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nb,n,crowded", [
    ((9, 7, 5), 630, False), ((9, 7, 5), 631, False),            # 315 cells: 256-cell groups, then 16
    ((40, 32, 16), 7, True), ((40, 32, 16), 900, False),         # groups of 128 particles and fewer load directly
    ((40, 32, 16), 2700, False), ((40, 32, 16), 40_000, True),   # and more; a crowded cell over many chunks
    ((16, 16, 32), 16_500, False), ((16, 16, 33), 17_000, True),   # groups of 16 and of 64
    ((40, 32, 16), 41_000, False), ((2, 3, 1), 3000, False), ((1, 1, 1), 2049, False), ((5, 4, 4), 5200, True)])
@pytest.mark.parametrize("precision", ["wide", "kahan", "naive", "fp64"])
def test_groups(nb, n, crowded, precision):
    import torch

    import paper_1807_11834_amd as cpl
    prec = {"wide": cpl.COUPLE_FP32_WIDE, "kahan": cpl.COUPLE_FP32_KAHAN, "naive": cpl.COUPLE_FP32_NAIVE,
            "fp64": cpl.COUPLE_FP64}[precision]
    dt = np.float64 if precision == "fp64" else np.float32
    u = 2.0 ** -53 if precision == "fp64" else 2.0 ** -24
    h = 1.0 / 64
    box = tuple(c * h for c in nb)
    rng = np.random.default_rng(n + nb[0])
    pos = rng.random((n, 3)) * box
    if crowded:   # two thirds in the last cell
        pos[: 2 * n // 3] = (np.array(nb) - rng.random((2 * n // 3, 3))) * h
    pos = pos.astype(dt)
    vel = rng.normal(size=(n, 3)).astype(dt)
    diam = (rng.uniform(0.05, 0.1, n) * h).astype(dt)
    fine = rng.normal(size=(4, 2 * nb[2], 2 * nb[1], 2 * nb[0])).astype(dt)
    cfg = cpl.Config(box=box, nb=nb, ratio=2, deposit=cpl.COUPLE_NGP, precision=prec, semi_implicit=1, eps_min=0.1,
                     vel_source=cpl.COUPLE_VEL_BULK, max_particles=n)
    put = lambda a: torch.from_numpy(a).to("cuda:0")
    print(f"case {nb} n{n} crowded={crowded} {precision}", flush=True)
    c = cpl.Coupler(cfg)
    out = c.step(put(pos), put(vel), put(diam), [put(f) for f in fine])
    g = {k: v.cpu().numpy().astype(np.float64) for k, v in out.items() if v is not None}
    d = cpl.diag_dict(out["diag"])
    c.close()
    ncell, vb = int(np.prod(nb)), h ** 3
    cell = g["cell"].astype(np.int64)
    most = np.bincount(cell, minlength=ncell).max()
    # terms of a cell: a few roundings each (product, volume), then of the sum: one for
    # each term where it is plain, a last one (and its residue) where it is not
    sums = 8 + (most if precision in ("naive", "fp64") else 2)
    gather = lambda v: np.bincount(cell, weights=v, minlength=ncell) / vb
    vol = np.pi / 6.0 * diam.astype(np.float64) ** 3
    beta, drag, v64 = g["beta"], g["drag"], vel.astype(np.float64)
    pairs = [(g["bulk_phi"].ravel(), gather(vol), gather(vol)), (g["bulk_K"].ravel(), gather(beta), gather(beta))]
    for a in range(3):
        pairs.append((g["bulk_F"].reshape(3, -1)[a], -gather(drag[:, a]), gather(np.abs(drag[:, a]))))
        pairs.append((g["bulk_KU"].reshape(3, -1)[a], gather(beta * v64[:, a]), gather(np.abs(beta * v64[:, a]))))
    for got, ref, mag in pairs:
        assert (np.abs(got - ref) <= sums * u * mag).all()
    # the pressure gradient does not depend on the deposition: the trilinear one's, bit for bit
    cfg.deposit = cpl.COUPLE_CIC
    c = cpl.Coupler(cfg)
    cic = c.step(put(pos), put(vel), put(diam), [put(f) for f in fine])
    assert torch.equal(out["bulk_G"], cic["bulk_G"])
    c.close()
    # FP64 sums of the cells' values: their order is free
    for name, field in (("V_dep", g["bulk_phi"]), ("K_b", g["bulk_K"])):
        assert abs(d[name] - field.sum() * vb) <= ncell * 2.0 ** -53 * np.abs(field).sum() * vb
    for a in range(3):
        f = g["bulk_F"].reshape(3, -1)[a]
        assert abs(d["S_b"][a] - f.sum() * vb) <= ncell * 2.0 ** -53 * np.abs(f).sum() * vb
    assert d["max_phi"] == g["bulk_phi"].max()
