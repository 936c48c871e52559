"""GPU: the fp32 tile kernel's inner products, which are formed from three bf16
slices of every value, against fp64: element by element, at the edges of tiles
and of staged blocks, for ordinary, one-signed and widely spread values, values
near the largest float and values whose lower slices are subnormal.

The prediction of a degree-1 polynomial model with alpha = e_j is the inner
product <x_j, x> as the kernel formed it in fp32."""
from __future__ import annotations

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _values(rng, kind, shape):
    x = rng.uniform(-1.0, 1.0, shape)
    if kind == "positive":
        x = np.abs(x)
    elif kind == "spread":
        x = x * np.exp(6.0 * rng.standard_normal(shape))
    elif kind == "huge":
        x = np.sign(x) * 3.4028234e38 * (1.0 - np.abs(x) * 2.0 ** -7)
    elif kind == "tiny":
        x = x * 2.0 ** -118
    elif kind == "subnormal":
        x = x * 2.0 ** -135
    return x.astype(np.float32)


# points at tile edges, features at the edges of 16- and 32-feature blocks
@pytest.mark.parametrize("n,nt,d", [(3, 1, 1), (127, 128, 15), (129, 5, 17), (256, 129, 33),
                                    (130, 200, 64), (150, 100, 1025)])
@pytest.mark.parametrize("kind", ["plain", "positive", "spread", "huge", "tiny", "subnormal"])
def test_inner_products_keep_fp32_accuracy(torch_dev, kind, n, nt, d):
    torch, dev = torch_dev
    import paper_2202_12674_amd as P
    rng = np.random.default_rng(1000 * d + n)
    A = _values(rng, kind, (n, d))
    # the other factor brings the products back into the range of floats
    other = {"huge": 2.0 ** -110, "tiny": 2.0 ** 60, "subnormal": 2.0 ** 100}.get(kind, 1.0)
    B = (_values(rng, kind if kind in ("positive", "spread") else "plain", (nt, d))
         * np.float32(other)).astype(np.float32)
    ref = A.astype(np.float64) @ B.astype(np.float64).T
    mag = np.abs(A.astype(np.float64)) @ np.abs(B.astype(np.float64)).T
    # three dropped products (2^-23), one ulp (2^-23) per sum of 16 features and
    # slice pair order, and the roundings of the joined sum and of the score
    tol = (4 + -(-d // 16)) * 2.0 ** -23 * mag
    Ad, Bd = torch.from_numpy(A).to(dev), torch.from_numpy(B).to(dev)
    for j in sorted({0, n // 2, n - 1}):
        e = torch.zeros(n, dtype=torch.float32, device=dev)
        e[j] = 1.0
        s, _ = P.predict(Ad, e, 0.0, Bd, kernel="poly", gamma=1.0, coef0=0.0, degree=1)
        err = np.abs(s.cpu().numpy().astype(np.float64) - ref[j])
        assert (err <= tol[j]).all(), (kind, j, float((err / tol[j]).max()))


@pytest.mark.parametrize("kernel,kw", [("poly", dict(gamma=2.0 ** 100, coef0=0.5, degree=2)),
                                       ("rbf", dict(gamma=2.0 ** 100)), ("linear", {})])
def test_products_and_training_on_tiny_points(torch_dev, kernel, kw):
    """Points around 2^-50 with a few entries down to the subnormals: the
    product against fp64 at the fp32 bar, and a training that converges to
    eps on it."""
    torch, dev = torch_dev
    import paper_2202_12674_amd as P
    rng = np.random.default_rng(5)
    n, d = 300, 40
    X = rng.uniform(-1.0, 1.0, (n, d)) * 2.0 ** -50
    X[::7, 3] *= 2.0 ** -70
    X = X.astype(np.float32)
    C = 2.0 ** 100 if kernel == "linear" else 1.0
    X64 = X.astype(np.float64)
    G = X64 @ X64.T
    if kernel == "poly":
        K = (kw["gamma"] * G + kw["coef0"]) ** 2
    elif kernel == "rbf":
        nrm = np.diag(G)
        K = np.exp(-kw["gamma"] * np.maximum(nrm[:, None] + nrm[None, :] - 2 * G, 0.0))
    else:
        K = G
    N = n - 1
    Q = K[:N, :N] - K[:N, N:] - K[N:, :N] + K[N, N] + 1.0 / C + np.eye(N) / C
    p = rng.standard_normal(N).astype(np.float32)
    Xd = torch.from_numpy(X).to(dev)
    out = P.matvec(Xd, torch.from_numpy(p).to(dev), C=C, kernel=kernel, **kw).double().cpu().numpy()
    ref = Q @ p.astype(np.float64)
    assert np.abs(out - ref).max() <= 1e-5 * np.abs(ref).max()
    y = np.where(rng.random(n) < 0.5, 1.0, -1.0).astype(np.float32)
    r = P.train(Xd, torch.from_numpy(y).to(dev), C=C, eps=1e-4, kernel=kernel, **kw)
    rhs = (y[:N] - y[N]).astype(np.float64)
    x = r.alpha.double().cpu().numpy()[:N]
    assert r.converged and np.linalg.norm(rhs - Q @ x) <= 1e-3 * np.linalg.norm(rhs)
