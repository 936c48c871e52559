"""GPU: the linear kernel's two passes over the points (w = X^T p, then X w) at
the edges of their launch shapes: odd and even feature counts (element-wise and
16-byte loads), points that are not 16-byte aligned, rows long enough to be
shared by four waves, few rows, the chunk and row-group remainders."""
from __future__ import annotations

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _reduced(X, C, p):
    N = len(X) - 1
    q = X[:N] @ X[N]
    qmm = X[N] @ X[N] + 1.0 / C
    return X[:N] @ (X[:N].T @ p) + (qmm - q) * p.sum() - q @ p + p / C


# above 2^17 values, so that no size takes the single-launch iteration
@pytest.mark.parametrize("n,d", [(2, 70000), (5, 40001), (33, 4100), (300, 1023), (1026, 128),
                                 (1030, 1024), (8193, 1024), (4097, 33), (70001, 3)])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("aligned", [True, False])
def test_product_prediction_and_training(torch_dev, n, d, dtype, aligned):
    torch, dev = torch_dev
    import paper_2202_12674_amd as P
    rng = np.random.default_rng(n + d)
    npd = np.float64 if dtype == "f64" else np.float32
    X = rng.uniform(-1.0, 1.0, (n, d)).astype(npd)
    buf = torch.zeros(n * d + 1, dtype=torch.from_numpy(X).dtype, device=dev)
    Xd = buf[0 if aligned else 1:][:n * d].view(n, d)
    Xd.copy_(torch.from_numpy(X))
    assert (Xd.data_ptr() % 16 == 0) == aligned
    X64 = X.astype(np.float64)
    p = rng.standard_normal(n - 1).astype(npd)
    out = P.matvec(Xd, torch.from_numpy(p).to(dev), C=3.0).double().cpu().numpy()
    ref = _reduced(X64, 3.0, p.astype(np.float64))
    # rounded once to the output type beside fp64 sums of n and d terms
    tol = (1e-13 if dtype == "f64" else 1.2e-7) * np.abs(ref).max()
    assert np.abs(out - ref).max() <= tol
    alpha = rng.standard_normal(n).astype(npd)
    Y = rng.uniform(-1.0, 1.0, (7, d)).astype(npd)
    s, lab = P.predict(Xd, torch.from_numpy(alpha).to(dev), 0.5, torch.from_numpy(Y).to(dev))
    f = Y.astype(np.float64) @ (X64.T @ alpha.astype(np.float64)) + 0.5
    assert np.abs(s.double().cpu().numpy() - f).max() <= \
        (1e-13 if dtype == "f64" else 1.2e-7) * max(1.0, np.abs(f).max()) * 4
    assert (lab.cpu().numpy() == np.where(s.cpu().numpy() > 0, 1, -1)).all()
    # three iterations of CG in numpy and on the device; the residual recurrence
    y = np.where(np.arange(n) % 3 == 0, -1.0, 1.0).astype(npd)
    k = min(3, n - 1)
    r = P.train(Xd, torch.from_numpy(y).to(dev), C=3.0, eps=1e-12, max_iter=k, history=4,
                true_residual=True)
    rhs = (y[:-1] - y[-1]).astype(np.float64)
    x, res = np.zeros(n - 1), rhs.copy()
    dv, rr = res.copy(), res @ res
    rr0, hist = rr, []
    for _ in range(r.iterations):
        q = _reduced(X64, 3.0, dv)
        a = rr / (dv @ q)
        x, res = x + a * dv, res - a * q
        rr, old = res @ res, rr
        hist.append(rr / rr0)
        dv = res + rr / old * dv
    assert np.allclose(r.history, hist, rtol=1e-6, atol=1e-20)
    got = r.alpha.double().cpu().numpy()
    assert np.abs(got[:-1] - x).max() <= (1e-8 if dtype == "f64" else 2e-7) * np.abs(x).max()


def test_nonfinite_points_leave_the_outputs_untouched(torch_dev):
    torch, dev = torch_dev
    import paper_2202_12674_amd as P
    X = torch.rand(3000, 101, dtype=torch.float64, device=dev)
    X[2999, 100] = float("inf")       # the pivot's last feature
    p = torch.rand(2999, dtype=torch.float64, device=dev)
    out = torch.full_like(p, 7.0)
    with pytest.raises(P.LssvmError) as e:
        P.matvec(X, p, out=out)
    assert e.value.code == -2 and bool((out == 7.0).all())
    y = torch.where(p > 0.5, 1.0, -1.0).to(p.dtype)
    with pytest.raises(P.LssvmError) as e:
        P.train(X, torch.cat([y, y[:1]]))
    assert e.value.code == -2


def _exact(a):
    from fractions import Fraction
    return [Fraction(float(v)) for v in a]


# four-wave rows with 16-byte and element-wise loads, a wave per four rows
@pytest.mark.parametrize("d", [2000, 1101, 300])
def test_scores_that_cancel_keep_the_pairs_bits(torch_dev, d):
    """Decision values whose terms cancel to their last bits, against exact
    rational sums. hi + lo holds every product's and every addition's error but
    for the roundings of lo itself: below (d + n) 2^-53 times what lo can hold,
    (d + n) 2^-53 sum |terms|. A sum that counts one error twice, or none, is
    off by 1e-18 of the terms or more."""
    torch, dev = torch_dev
    import paper_2202_12674_amd as P
    rng = np.random.default_rng(d)
    n = 3
    X, alpha = rng.standard_normal((n, d)), rng.standard_normal(n)
    w = [sum(a * x for a, x in zip(_exact(alpha), _exact(X[:, k]))) for k in range(d)]
    Y = rng.standard_normal((9, d))
    ref, mag = [], []
    for t in range(9):
        head = sum(y * v for y, v in zip(_exact(Y[t, :-1]), w))
        Y[t, -1] = float(-head / w[-1])
        terms = [y * v for y, v in zip(_exact(Y[t]), w)]
        ref.append(sum(terms))
        mag.append(float(sum(abs(v) for v in terms)))
    s, _ = P.predict(*(torch.from_numpy(v).to(dev) for v in (X, alpha)), 0.0,
                     torch.from_numpy(Y).to(dev))
    for t, got in enumerate(_exact(s.cpu().numpy())):
        bar = ((d + n) * 2.0 ** -53) ** 2 * mag[t] + 2.0 ** -52 * abs(float(ref[t]))
        assert abs(float(got - ref[t])) <= bar, (t, float(got - ref[t]) / mag[t])


def test_weights_that_cancel_keep_the_pairs_bits(torch_dev):
    """The same over the points: w_0 = sum alpha_i x_i0 cancels, over many chunks
    of rows; the score of e_0 is w_0."""
    torch, dev = torch_dev
    import paper_2202_12674_amd as P
    rng = np.random.default_rng(4)
    n, d = 4001, 5
    X, alpha = rng.standard_normal((n, d)), rng.standard_normal(n)
    x0, a = _exact(X[:, 0]), _exact(alpha)
    alpha[-1] = float(-sum(u * v for u, v in zip(x0[:-1], a[:-1])) / x0[-1])
    terms = [u * v for u, v in zip(x0, _exact(alpha))]
    Y = np.eye(1, d)
    s, _ = P.predict(*(torch.from_numpy(v).to(dev) for v in (X, alpha)), 0.0,
                     torch.from_numpy(Y).to(dev))
    bar = ((d + n) * 2.0 ** -53) ** 2 * float(sum(map(abs, terms))) + \
        2.0 ** -52 * abs(float(sum(terms)))
    assert abs(float(_exact(s.cpu().numpy())[0] - sum(terms))) <= bar


@pytest.mark.parametrize("d", [5, 2000])
def test_scores_that_overflow_are_infinite(torch_dev, d):
    """An infinite coefficient, or values whose products overflow, give infinite
    scores of the plain sums' sign, not NaN."""
    torch, dev = torch_dev
    import paper_2202_12674_amd as P
    X = torch.rand(40, d, dtype=torch.float64, device=dev) + 0.5
    Y = torch.rand(6, d, dtype=torch.float64, device=dev) + 0.5
    Y[3:] *= -1.0
    for a, scale in ((float("inf"), 1.0), (1e200, 1e200)):
        alpha = torch.full((40,), 1.0, dtype=torch.float64, device=dev)
        alpha[17] = a
        s, lab = P.predict(X * scale, alpha, 0.5, Y)
        assert s.tolist() == [float("inf")] * 3 + [-float("inf")] * 3
        assert lab.tolist() == [1] * 3 + [-1] * 3
