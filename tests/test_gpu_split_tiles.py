"""GPU: polynomial and RBF products whose tiles are shared over several
workgroups in unequal shares (few tiles of many features, and in fp64 the tiles
left after the last full round of one per CU), against fp64, and trainings on
them whose residual is checked with the explicit matrix."""
from __future__ import annotations

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _reduced(kernel, X, C, gamma):
    G = X @ X.T
    if kernel == "poly":
        K = (gamma * G + 1.0) ** 3
    else:
        nrm = np.diag(G)
        K = np.exp(-gamma * np.maximum(nrm[:, None] + nrm[None, :] - 2 * G, 0.0))
    N = len(X) - 1
    return K[:N, :N] - K[:N, N:] - K[N:, :N] + K[N, N] + 1.0 / C + np.eye(N) / C


# (one tile, uneven shares; three; fused trainings, the last of 4 rows a thread and
# the first and last of 8; the first not fused; 351 and 300 tiles: 95 and 44 of
# them split in fp64; 136 tiles in 408 shares in fp64, 253 left whole)
@pytest.mark.parametrize("n,d", [(2, 5000), (129, 1100), (257, 333), (502, 2877), (907, 1100),
                                 (1025, 700), (1026, 40), (1400, 1000), (2049, 70),
                                 (2050, 300), (3300, 800), (3000, 513), (2040, 420), (2800, 260)])
@pytest.mark.parametrize("kernel,dtype", [("poly", "f64"), ("rbf", "f32"), ("rbf", "f64"),
                                          ("poly", "f32")])
def test_product_and_training(torch_dev, kernel, dtype, n, d):
    torch, dev = torch_dev
    import paper_2202_12674_amd as P
    rng = np.random.default_rng(n + d)
    npd = np.float64 if dtype == "f64" else np.float32
    X = rng.uniform(-1.0, 1.0, (n, d)).astype(npd)
    Q = _reduced(kernel, X.astype(np.float64), 2.0, 1.0 / d)
    Xd = torch.from_numpy(X).to(dev)
    kw = dict(kernel=kernel, gamma=1.0 / d, coef0=1.0, degree=3, C=2.0)
    bar = 1e-11 if dtype == "f64" else 1e-5
    for seed in range(2):
        p = rng.standard_normal(n - 1).astype(npd)
        out = P.matvec(Xd, torch.from_numpy(p).to(dev), **kw).double().cpu().numpy()
        ref = Q @ p.astype(np.float64)
        assert np.abs(out - ref).max() <= bar * np.abs(ref).max()
    y = np.where(rng.random(n) < 0.5, 1.0, -1.0).astype(npd)
    y[0], y[-1] = 1.0, -1.0
    eps = 1e-9 if dtype == "f64" else 1e-5
    r = P.train(Xd, torch.from_numpy(y).to(dev), eps=eps, **kw)
    again = P.train(Xd, torch.from_numpy(y).to(dev), eps=eps, **kw)
    assert r.converged and torch.equal(r.alpha, again.alpha)
    rhs = (y[:-1] - y[-1]).astype(np.float64)
    x = r.alpha.double().cpu().numpy()[:-1]
    assert np.linalg.norm(rhs - Q @ x) <= (2 * eps if dtype == "f64" else 30 * eps) * \
        np.linalg.norm(rhs)
