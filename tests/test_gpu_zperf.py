"""Throughput floor of the implicit product: a change that keeps every result
right but loses a large share of the matrix-core rate fails here. The floors
are 70% of the published fp64 peak (the product runs at 93-94% of it) and, for
fp32 on the bf16 matrix cores, 160 TFLOP/s (it runs at 208-225), far enough
below to hold on any healthy board. Collected last, so a slow
board cannot hide a parity failure behind it."""
from __future__ import annotations

import pytest

import synthdata as S

FLOOR_TFLOPS = {"f64": 0.70 * 78.6, "f32": 160.0}


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    import paper_2202_12674_amd as P
    P.lib()  # fail loudly if the HIP library is missing
    return torch, torch.device("cuda:0")


@pytest.mark.gpu
@pytest.mark.parametrize("kernel,dtype,n,d", [("poly", "f32", 16384, 4096),
                                              ("rbf", "f64", 16384, 2048)])
def test_product_rate_floor(torch_dev, kernel, dtype, n, d):
    torch, dev = torch_dev
    import paper_2202_12674_amd as P
    kp = dict(poly=dict(gamma=1.0 / d, coef0=1.0, degree=3), rbf=dict(gamma=1.0 / d))[kernel]
    cfg = S.Config(f"{kernel}_{dtype}_{n}x{d}", dtype, kernel, n, d, mu=1.0, inf_frac=0.3,
                   flip_frac=0.05, C=1.0, eps=1e-3, **kp)
    X, y, _ = S.make_train(cfg)
    Xd, yd = torch.from_numpy(X).to(dev), torch.from_numpy(y).to(dev)
    kw = dict(kernel=kernel, gamma=cfg.gamma, coef0=cfg.coef0, degree=cfg.degree)
    P.train(Xd, yd, C=cfg.C, eps=cfg.eps, **kw)   # warm-up
    r = P.train(Xd, yd, C=cfg.C, eps=cfg.eps, time_matvec=True, matvec_times=256, **kw)
    assert r.converged and len(r.matvec_times) >= 3
    ms = sorted(r.matvec_times)[len(r.matvec_times) // 2]
    N = n - 1
    rate = N * (N + 1) * d / (ms * 1e-3) / 1e12
    print(f"{cfg.name}: {ms:.3f} ms per product, {rate:.1f} TFLOP/s", flush=True)
    assert rate >= FLOOR_TFLOPS[dtype], f"{cfg.name}: {rate:.1f} TFLOP/s"


@pytest.mark.gpu
def test_one_tiny_value_costs_a_layout_not_a_product(torch_dev):
    """A value whose slices would be subnormal has an fp32 model laid out anew,
    scaled up: the product and the scores wait for that instead of running twice."""
    torch, dev = torch_dev
    import paper_2202_12674_amd as P
    n, d = 32768, 1024
    g = torch.Generator(device=dev)
    g.manual_seed(1)
    X = torch.rand(n, d, generator=g, device=dev) * 2 - 1
    v = torch.randn(n, generator=g, device=dev)
    Y = X[:2048] * 0.5
    ws = P.alloc_workspace(max(P.workspace_bytes(n, d, X.dtype),
                               P.predict_workspace_bytes(n, 2048, d, X.dtype)), dev)

    def ms(f):
        f()
        times = []
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            f()
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b))
        return sorted(times)[2]

    kw = dict(kernel="rbf", gamma=1.0 / d, workspace=ws)
    calls = [lambda: P.matvec(X, v[:-1], **kw), lambda: P.predict(X, v, 0.0, Y, **kw)]
    plain = [ms(f) for f in calls]
    X[77, 3] = 1e-37
    tiny = [ms(f) for f in calls]
    print(f"product and scores: {plain} ms, with a tiny value {tiny} ms", flush=True)
    assert tiny[0] <= 1.35 * plain[0] and tiny[1] <= 1.6 * plain[1]
