"""GPU: decision values of up to 128 points straight from the caller's rows
(polynomial and RBF models) against fp64, at the edges of its blocks of 16 and
32 model points, of 16 to 128 test points and of 16-feature chunks, with points
that are not 16-byte aligned; 129 points (the tile path) beside them; values
that are not finite."""
from __future__ import annotations

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _decision(kernel, X, a, Y, gamma, coef0, degree):
    G = Y @ X.T
    if kernel == "poly":
        return (gamma * G + coef0) ** degree @ a
    dist = (Y * Y).sum(1)[:, None] + (X * X).sum(1)[None, :] - 2 * G
    return np.exp(-gamma * np.maximum(dist, 0.0)) @ a


@pytest.mark.parametrize("n,nt,d", [(1, 1, 1), (15, 16, 3), (16, 17, 16), (33, 32, 17),
                                    (2049, 33, 100), (31, 64, 257), (40000, 65, 20),
                                    (1000, 128, 65), (300, 129, 65), (20000, 2, 1),
                                    (8192, 100, 20), (8193, 100, 20), (16385, 65, 33),
                                    (8193, 70, 512)])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("kernel", ["poly", "rbf"])
def test_scores_and_labels(torch_dev, kernel, dtype, n, nt, d):
    torch, dev = torch_dev
    import paper_2202_12674_amd as P
    rng = np.random.default_rng(n + nt + d)
    npd = np.float64 if dtype == "f64" else np.float32
    X, Y = (rng.uniform(-1.0, 1.0, (k, d)).astype(npd) for k in (n, nt))
    a = rng.standard_normal(n).astype(npd)
    kw = dict(gamma=1.0 / d, coef0=0.5, degree=3)
    args = [v.astype(np.float64) for v in (X, a, Y)]
    f = _decision(kernel, *args, **kw) + 0.25
    # kernel values of d + 20 roundings each, relative to values up to 1.5^3
    u = 2.0 ** -53 if dtype == "f64" else 2.0 ** -24
    tol = (d + 40) * u * (np.abs(a.astype(np.float64)).sum() * 4 + 1)
    for shift in (0, 1):
        def put(v):
            buf = torch.zeros(v.size + shift, dtype=torch.from_numpy(v).dtype, device=dev)
            buf[shift:] = torch.from_numpy(v.reshape(-1))
            return buf[shift:].view(*v.shape)
        s, lab = P.predict(put(X), put(a), 0.25, put(Y), kernel=kernel, **kw)
        got = s.double().cpu().numpy()
        assert np.abs(got - f).max() <= tol, (np.abs(got - f).max(), tol)
        sure = np.abs(f) > tol
        assert (lab.cpu().numpy()[sure] == np.where(f > 0, 1, -1)[sure]).all()


@pytest.mark.parametrize("where", ["train", "test"])
def test_nonfinite_values_leave_the_outputs_untouched(torch_dev, where):
    torch, dev = torch_dev
    import ctypes
    import paper_2202_12674_amd as P
    from paper_2202_12674_amd import _binding as B
    X = torch.rand(500, 9, dtype=torch.float64, device=dev)
    Y = torch.rand(5, 9, dtype=torch.float64, device=dev)
    (X if where == "train" else Y)[-1, -1] = float("inf")
    a = torch.rand(500, dtype=torch.float64, device=dev)
    s = torch.full((5,), 7.0, dtype=torch.float64, device=dev)
    ws = P.alloc_workspace(P.predict_workspace_bytes(500, 5, 9, X.dtype), dev)
    kp = B.Params(0.1, 1.0, 2)
    p = [ctypes.c_void_p(t.data_ptr()) for t in (X, a, Y, ws, s)]
    code = P.lib().lssvm_predict(p[0], p[1], 0.0, 500, 9, 0, 1, ctypes.byref(kp), p[2], 5, p[3],
                                 ws.numel(), p[4], None, None)
    assert code == B.ENONFINITE and bool((s == 7.0).all())


@pytest.mark.parametrize("nt", [5, 128, 129])
def test_fp32_polynomial_values_are_formed_in_fp64(torch_dev, nt):
    """Inner products that fp32 holds exactly: what is left is the rounding of
    the score, 2^-24, whichever path the number of points takes (the base and
    the power in fp32 would add their own)."""
    torch, dev = torch_dev
    import paper_2202_12674_amd as P
    rng = np.random.default_rng(nt)
    X, Y = (rng.integers(0, 4, (k, 20)).astype(np.float32) for k in (40, nt))
    a = rng.integers(1, 5, 40).astype(np.float32)
    kw = dict(gamma=0.1, coef0=0.3, degree=7)
    f = _decision("poly", *(v.astype(np.float64) for v in (X, a, Y)), **kw)
    s, _ = P.predict(*(torch.from_numpy(v).to(dev) for v in (X, a)), 0.0,
                     torch.from_numpy(Y).to(dev), kernel="poly", **kw)
    assert (np.abs(s.double().cpu().numpy() - f) <= 2.0 ** -24 * (1 + 1e-6) * f).all()
