"""Batch inference at the edges of its 16-row tiles and 256-row groups, on unaligned
features and into an output that overlaps them: every row against the oracle
network once, then bit for bit the same whatever the batch around it."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

ROWS = 256 * 256 * 2 + 300      # more groups than a 256-unit chip takes at once


@pytest.fixture(scope="module")
def net():
    import paper_1807_11834_amd as cpl
    from oracle import mlp as M
    rng = np.random.default_rng(5)
    feat = (rng.normal(size=(ROWS, 193)) * 0.3 + 1.0).astype(np.float32)
    params = M.init_params(3)
    mean, std = M.norm_stats(feat[:5000].astype(np.float64))
    m = cpl.Mlp(ROWS)
    m.set_params(M.flatten(params))
    m.set_norm(mean, std, np.ones(3))
    X = torch.from_numpy(feat).cuda()
    y = torch.empty((ROWS, 3), device="cuda")
    m.forward(X, y)
    at = np.r_[0:400, ROWS - 400:ROWS]
    ref, _ = M.forward(params, M.standardise(feat[at].astype(np.float64), mean, std), emulate=True)
    got = y.cpu().numpy()[at]
    # the tolerances of the network's parity tests: norm-wise 1e-3, each row 1e-2
    assert np.linalg.norm(got - ref) <= 1e-3 * np.linalg.norm(ref)
    rms = np.sqrt((ref ** 2).sum(1).mean())
    assert (np.linalg.norm(got - ref, axis=1) <= 1e-2 * np.maximum(np.linalg.norm(ref, axis=1), 1e-2 * rms)).all()
    yield m, X, y
    m.close()


@pytest.mark.parametrize("n", [1, 15, 16, 17, 31, 32, 33, 255, 256, 257, 8191, 65536, 65537])
def test_rows(net, n):
    m, X, y = net
    out = torch.full((n + 1, 3), 7.0, device="cuda")
    m.forward(X[:n], out[:n])
    assert torch.equal(out[:n], y[:n])
    assert bool((out[n] == 7.0).all())


def test_unaligned_and_overlapping(net):
    m, X, y = net
    n = 700
    pool = torch.empty(193 * n + 3, device="cuda")
    feat = pool[1:1 + 193 * n].view(n, 193)
    feat.copy_(X[:n])
    out = torch.empty(3 * n + 1, device="cuda")[1:].view(n, 3)
    m.forward(feat, out)
    assert torch.equal(out, y[:n])
    inside = pool[193 * 100:193 * 100 + 3 * n].view(n, 3)     # inside the features
    m.forward(feat, inside)
    assert torch.equal(inside, y[:n])
