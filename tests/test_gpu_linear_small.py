"""GPU: linear trainings that run whole in one workgroup (the points fit its
LDS) against the oracle and against the same training by separate launches (a
warm start from zeros takes those): lane groups of 1 to 16 threads per row and
per column, ragged remainders, residual recomputations, every end of CG."""
from __future__ import annotations

import numpy as np
import pytest

import oracle as O
import synthdata as S
from gpu_common import check_train, kw_of, oracle_ref, small_cfg, spec_of, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,n,d", [("f64", 2, 3), ("f64", 3, 5000), ("f64", 65, 33),
                                       ("f64", 129, 100), ("f64", 256, 64), ("f64", 1000, 16),
                                       ("f64", 1024, 9), ("f32", 257, 65), ("f32", 513, 40),
                                       ("f32", 1024, 24), ("f32", 17, 1025)])
def test_matches_the_oracle_and_separate_launches(torch_dev, dtype, n, d):
    torch, dev = torch_dev
    import paper_2202_12674_amd as P
    cfg = small_cfg("linear", dtype, n, d, C=1.0)
    X, y, _ = S.make_train(cfg)
    res = check_train(torch, dev, cfg, oracle_ref(cfg, X, y), X, y)
    Xd, yd = to_dev(torch, dev, X), to_dev(torch, dev, y)
    sep = P.train(Xd, yd, C=cfg.C, eps=cfg.eps, alpha0=torch.zeros_like(yd), **kw_of(cfg))
    assert abs(sep.iterations - res.iterations) <= max(2, res.iterations // 10)
    scale = float(sep.alpha.abs().max())
    assert float((sep.alpha - res.alpha).abs().max()) <= (1e-8 if dtype == "f64" else 1e-4) * scale
    again = P.train(Xd, yd, C=cfg.C, eps=cfg.eps, **kw_of(cfg))
    assert torch.equal(again.alpha, res.alpha) and again.b == res.b


def test_recomputations_history_and_caps(torch_dev):
    torch, dev = torch_dev
    import paper_2202_12674_amd as P
    cfg = small_cfg("linear", "f64", 200, 80, C=100.0)
    X, y, _ = S.make_train(cfg)
    Xd, yd = to_dev(torch, dev, X), to_dev(torch, dev, y)
    Qt, _, _ = O.reduced_matrix(X, spec_of(cfg), cfg.C)
    rhs = O.reduced_rhs(y)
    ref = O.solve_cg(lambda v: Qt @ v, rhs, 1e-10)
    r = P.train(Xd, yd, C=cfg.C, eps=1e-10, history=1000, true_residual=True)
    assert r.converged and r.iterations > 50          # past a recomputation
    assert abs(r.iterations - ref.iterations) <= max(2, ref.iterations // 10)
    assert len(r.history) == min(r.iterations, 257) and r.n_matvec == r.iterations + r.iterations // 50
    assert r.true_rel_residual <= 2e-10
    cap = P.train(Xd, yd, C=cfg.C, eps=1e-10, max_iter=7)
    assert cap.status == 1 and cap.iterations == 7 and not cap.stalled
    low = P.train(Xd, yd, C=cfg.C, eps=1e-15, max_iter=5000, true_residual=True)
    assert low.converged or low.stalled
    assert low.true_rel_residual <= 1e-11
    same = P.train(Xd, torch.ones_like(yd), C=cfg.C, eps=1e-10)
    assert same.iterations == 0 and same.b == 1.0 and bool((same.alpha == 0).all())


@pytest.mark.parametrize("what", ["point", "label"])
def test_bad_inputs_are_reported(torch_dev, what):
    torch, dev = torch_dev
    import paper_2202_12674_amd as P
    X = torch.rand(100, 7, dtype=torch.float64, device=dev)
    y = torch.where(torch.rand(100, device=dev) > 0.5, 1.0, -1.0).to(X.dtype)
    if what == "point":
        X[99, 6] = float("nan")
    else:
        y[98] = 0.5
    with pytest.raises(P.LssvmError) as e:
        P.train(X, y)
    assert e.value.code == (-2 if what == "point" else -3)


def test_nothing_to_solve_beside_overflowing_values(torch_dev):
    """Equal labels end before the first iteration whatever q holds: alpha = 0 in
    every run, also where q_i overflows (b is then NaN, as 0 times it is)."""
    torch, dev = torch_dev
    import paper_2202_12674_amd as P
    X = torch.rand(256, 64, dtype=torch.float64, device=dev) + 0.5
    y = torch.ones(256, dtype=torch.float64, device=dev)
    for scale in (1.0, 1e200):
        for _ in range(20):
            r = P.train(X * scale, y, C=1.0, eps=1e-10)
            assert r.converged and r.iterations == 0 and bool((r.alpha == 0).all())
            assert r.b == 1.0 if scale == 1.0 else np.isnan(r.b)
