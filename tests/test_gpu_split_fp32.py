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


KINDS = ["plain", "positive", "spread", "huge", "tiny", "subnormal"]


# points at tile edges, features at the edges of 16- and 32-feature blocks; more than
# 128 test points, which tiles take
@pytest.mark.parametrize("n,nt,d", [(3, 129, 1), (127, 130, 15), (129, 129, 17), (256, 129, 33),
                                    (130, 200, 64), (150, 129, 1025)])
@pytest.mark.parametrize("kind", KINDS)
def test_inner_products_keep_fp32_accuracy(torch_dev, kind, n, nt, d):
    # three dropped products (2^-23), one ulp (2^-23) per sum of 16 features and
    # slice pair order, and the roundings of the joined sum and of the score
    _check_inner_products(torch_dev, kind, n, nt, d, (4 + -(-d // 16)) * 2.0 ** -23)


# the fp32 instruction of few test points, straight from the rows
@pytest.mark.parametrize("n,nt,d", [(3, 1, 1), (127, 128, 15), (129, 5, 17), (150, 100, 1025)])
@pytest.mark.parametrize("kind", KINDS)
def test_inner_products_of_few_points_keep_fp32_accuracy(torch_dev, kind, n, nt, d):
    # half an ulp for each product and each addition of a wave's quarter of the
    # features, for the three additions of the waves' sums and for the score
    _check_inner_products(torch_dev, kind, n, nt, d, (8 + -(-d // 2)) * 2.0 ** -24)


def _check_inner_products(torch_dev, kind, n, nt, d, rel):
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
    tol = rel * mag
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


# the smallest inner products that fp32 holds in full, and some below
@pytest.mark.parametrize("exponent", [52, 56, 58, 60, 62, 70])
@pytest.mark.parametrize("n,nt,d", [(130, 200, 1), (130, 129, 3), (256, 200, 40)])
def test_small_values_keep_fp32_accuracy(torch_dev, exponent, n, nt, d):
    """Points around 2^-exponent: the products of lower slices lie far below the
    smallest normal float long before x y does. gamma brings the values back."""
    torch, dev = torch_dev
    import paper_2202_12674_amd as P
    rng = np.random.default_rng(d + exponent)
    A, B = ((rng.uniform(-1.0, 1.0, (k, d)) * 2.0 ** -exponent).astype(np.float32)
            for k in (n, nt))
    gamma = 2.0 ** (2 * exponent)
    ref = gamma * (A.astype(np.float64) @ B.astype(np.float64).T)
    mag = gamma * (np.abs(A.astype(np.float64)) @ np.abs(B.astype(np.float64)).T)
    tol = (4 + -(-d // 16)) * 2.0 ** -23 * mag   # as above
    Ad, Bd = torch.from_numpy(A).to(dev), torch.from_numpy(B).to(dev)
    for j in range(0, n, 13):
        e = torch.zeros(n, dtype=torch.float32, device=dev)
        e[j] = 1.0
        s, _ = P.predict(Ad, e, 0.0, Bd, kernel="poly", gamma=gamma, coef0=0.0, degree=1)
        err = np.abs(s.cpu().numpy().astype(np.float64) - ref[j])
        assert (err <= tol[j]).all(), (j, float((err / tol[j]).max()))


@pytest.mark.parametrize("low,high", [(-75, 10), (-40, 35), (-40, 45), (-120, 0), (-60, 60)])
def test_values_of_any_range_by_the_products(torch_dev, low, high):
    """Values spread over 2^low .. 2^high (the stored scale is chosen by the range):
    RBF products and degree-1 products against fp64, a training to eps. gamma makes
    the largest values' distances about 1."""
    torch, dev = torch_dev
    import paper_2202_12674_amd as P
    rng = np.random.default_rng(high - low)
    n, d = 300, 21
    X = rng.uniform(-1.0, 1.0, (n, d)) * 2.0 ** high
    X[:, 1::2] *= 2.0 ** rng.uniform(low - high, 0.0, (n, len(range(1, d, 2))))
    X = X.astype(np.float32)
    X64, N = X.astype(np.float64), n - 1
    G = X64 @ X64.T
    gamma = 2.0 ** (-2 * high) / d
    nrm = np.diag(G)
    K = {"rbf": np.exp(-gamma * np.maximum(nrm[:, None] + nrm[None, :] - 2 * G, 0.0)),
         "poly": gamma * G + 0.5}
    Xd = torch.from_numpy(X).to(dev)
    p = rng.standard_normal(N).astype(np.float32)
    y = np.where(rng.random(n) < 0.5, 1.0, -1.0).astype(np.float32)
    for kernel, k in K.items():
        kw = dict(kernel=kernel, gamma=gamma, coef0=0.5, degree=1, C=1.0)
        Q = k[:N, :N] - k[:N, N:] - k[N:, :N] + k[N, N] + 1.0 + np.eye(N)
        out = P.matvec(Xd, torch.from_numpy(p).to(dev), **kw).double().cpu().numpy()
        ref = Q @ p.astype(np.float64)
        assert np.abs(out - ref).max() <= 1e-5 * np.abs(ref).max(), kernel
        r = P.train(Xd, torch.from_numpy(y).to(dev), eps=1e-5, **kw)
        rhs = (y[:N] - y[N]).astype(np.float64)
        x = r.alpha.double().cpu().numpy()[:N]
        assert r.converged and np.linalg.norm(rhs - Q @ x) <= 1e-4 * np.linalg.norm(rhs), kernel
