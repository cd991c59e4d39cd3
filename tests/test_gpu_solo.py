"""Solves of small windows (whole epochs in one workgroup) against the oracle."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_1206_6409_amd import gencd as G
from paper_1206_6409_amd import synth

pytestmark = pytest.mark.gpu

RULES = {"cyclic": O.CYCLIC, "stochastic": O.STOCHASTIC, "shotgun": O.SHOTGUN}


def _solve_both(P, rule, S, epochs, tol=0.0, check_every=1, lam_ratio=0.1, w0=None):
    Xo = O.Matrix.of(P)
    lam = lam_ratio * O.lambda_max(Xo, P.y, P.loss)
    ref = O.solve(Xo, P.y, P.loss, lam, RULES[rule], select_size=S, seed=9, tol=tol,
                  max_epochs=epochs, check_every=check_every,
                  w0=None if w0 is None else w0.astype(np.float64))
    X = G.Matrix.of(P)
    prm = G.make_params(P.loss, lam, rule=rule, select_size=S, seed=9, tol=tol, max_epochs=epochs,
                        check_every=check_every)
    res = G.solve(X, torch.as_tensor(P.y, device="cuda"), prm,
                  w0=None if w0 is None else torch.as_tensor(w0, device="cuda"))
    return ref, res


def _bound(P, epochs):
    """A column of L entries forms its step from L FP32 products and sums of
    a residual that is itself rounded: an error of about 2 L 2^-24 of
    sum |x r| / (beta sum x^2), at most 8 L 2^-24 max|r| for N(0, 1) values
    (beta >= 1/4), added once per epoch."""
    lmax = int(np.diff(P.col_ptr).max())
    r = 1.0 if P.loss == synth.LOGISTIC else float(np.abs(P.y).max())
    return epochs * 8.0 * lmax * 2.0**-24 * max(1.0, r)


# edges of the shapes: one wave (S <= 4), more columns than groups, columns
# longer than the first batch, a last window that is nearly empty, more rows
# than fit the in-launch check or LDS, more entries than the in-launch check
# takes, more windows than one launch runs
@pytest.mark.parametrize("n,k,density,loss,rule,S", [
    (400, 1000, 0.01, synth.LOGISTIC, "cyclic", 1),
    (400, 1000, 0.01, synth.SQUARED, "stochastic", 1),
    (300, 500, 0.3, synth.LOGISTIC, "cyclic", 1),
    (400, 1000, 0.01, synth.LOGISTIC, "shotgun", 3),
    (400, 1001, 0.01, synth.LOGISTIC, "shotgun", 5),
    (400, 1000, 0.01, synth.SQUARED, "shotgun", 128),
    (400, 1000, 0.01, synth.LOGISTIC, "shotgun", 129),
    (400, 1000, 0.01, synth.LOGISTIC, "shotgun", 333),
    (60, 70, 0.05, synth.LOGISTIC, "shotgun", 7),
    (200, 300, 0.2, synth.SQUARED, "shotgun", 9),
    (900, 400, 0.1, synth.LOGISTIC, "shotgun", 16),
    (7900, 300, 0.002, synth.LOGISTIC, "shotgun", 24),
    (9000, 300, 0.002, synth.SQUARED, "shotgun", 24),
    (13400, 300, 0.001, synth.LOGISTIC, "shotgun", 24),
    (3000, 5000, 0.01, synth.LOGISTIC, "shotgun", 40),
    (300, 18000, 0.01, synth.LOGISTIC, "cyclic", 1),
])
def test_epochs_match_the_oracle(n, k, density, loss, rule, S):
    P = synth.make_bernoulli_problem(n, k, density, loss, seed=n + k, support=10)
    epochs = 2
    ref, res = _solve_both(P, rule, S, epochs)
    assert res.stats["epochs"] == ref.epochs and res.stats["iters"] == ref.iters
    err = np.abs(res.w.cpu().numpy().astype(np.float64) - ref.w).max()
    assert err <= _bound(P, epochs) * max(1.0, np.abs(ref.w).max()), err


@pytest.mark.parametrize("check_every", [1, 3, 0, -2])
def test_stops_at_the_oracles_epoch(check_every):
    P = synth.c1_ccd_logistic(scale=0.2)
    ref, res = _solve_both(P, "shotgun", 64, 500, tol=1e-6, check_every=max(check_every, 1))
    if check_every > 0:
        assert res.stats["epochs"] == ref.epochs
    assert res.status == G.OK and res.stats["kkt_max"] <= 1e-6
    assert abs(res.stats["objective"] - ref.objective) <= 1e-6 * abs(ref.objective)
    chk = O.check(O.Matrix.of(P), P.y, P.loss, 0.1 * O.lambda_max(O.Matrix.of(P), P.y, P.loss),
                  res.w.cpu().numpy().astype(np.float64))
    assert abs(chk.kkt - res.stats["kkt_max"]) <= 1e-9
    assert chk.nnz_w == res.stats["nnz_w"]


def test_warm_start():
    P = synth.make_bernoulli_problem(300, 800, 0.05, synth.SQUARED, seed=4, support=10)
    w0 = np.random.default_rng(0).standard_normal(P.k).astype(np.float32) * 0.01
    ref, res = _solve_both(P, "shotgun", 20, 2, w0=w0)
    err = np.abs(res.w.cpu().numpy().astype(np.float64) - ref.w).max()
    assert err <= _bound(P, 2) * max(1.0, np.abs(ref.w).max())


def test_divergence_guard_halves_the_window():
    """Five columns on one row overshoot together; the guard restores the
    last checked point and halves |J|, exactly as on the kernels that an
    explicit schedule selects."""
    P = synth.make_bernoulli_problem(1, 5, 1.0, synth.SQUARED, seed=6, support=10)
    X, y = G.Matrix.of(P), torch.as_tensor(P.y, device="cuda")
    lam = 0.1 * G.lambda_max(X, y, P.loss)
    kw = dict(rule="shotgun", select_size=5, seed=9, tol=1e-6, max_epochs=60)
    a = G.solve(X, y, G.make_params(P.loss, lam, **kw))
    b = G.solve(X, y, G.make_params(P.loss, lam, group=8, piece=256, **kw))
    assert a.stats["select_size"] < 5
    for key in ("select_size", "epochs", "iters", "coord_updates", "converged"):
        assert a.stats[key] == b.stats[key], key
    assert abs(a.stats["objective"] - b.stats["objective"]) <= 1e-6 * abs(b.stats["objective"])
