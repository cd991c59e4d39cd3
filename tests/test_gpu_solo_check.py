"""The FP64 checks that a small solve runs in its own launch agree with the
separate kernels' (an explicit schedule, and gencd_check) on weights of
columns without entries, on a NaN and on the drift of every check."""
import math

import numpy as np
import pytest
import torch

from paper_1206_6409_amd import gencd as G
from paper_1206_6409_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("count", [1, 3])
def test_weights_of_empty_columns_count(count):
    """A nonzero weight on a column without entries never moves and violates
    the optimality conditions by lambda."""
    P = synth.make_bernoulli_problem(400, 1000, 0.002, synth.LOGISTIC, seed=3, support=10)
    empty = np.nonzero(np.diff(P.col_ptr) == 0)[0]
    w0 = np.zeros(P.k, np.float32)
    w0[empty[5:5 + count]] = [5.0, -0.5, 1e-3][:count]
    X, y = G.Matrix.of(P), torch.as_tensor(P.y, device="cuda")
    lam = 0.1 * G.lambda_max(X, y, P.loss)
    kw = dict(rule="shotgun", select_size=20, seed=9, tol=1e-6, max_epochs=40)
    w0 = torch.as_tensor(w0, device="cuda")
    res = [G.solve(X, y, G.make_params(P.loss, lam, **kw, **sched), w0=w0)
           for sched in ({}, dict(group=8, piece=256))]
    chk = G.check(X, y, P.loss, lam, res[0].w)
    st = res[0].stats
    assert res[0].status == res[1].status == G.NOT_CONVERGED and not st["converged"]
    assert st["epochs"] == res[1].stats["epochs"] == 40
    assert st["nnz_w"] == chk.nnz_w >= count
    # the same FP64 sums in another order
    for got, want in ((st["kkt_max"], chk.kkt), (st["objective"], chk.objective),
                      (st["gap"], chk.gap)):
        assert abs(got - want) <= 1e-12 * max(1.0, abs(want))
    assert abs(st["kkt_max"] - lam) <= 1e-12


# the NaN's column decides the lane, the group and the round that meet it
@pytest.mark.parametrize("at", [0, 1, 6, 17, 63, 200, 511, 799])
def test_a_nan_gradient_is_not_optimal(at):
    """A NaN entry: the column has no curvature and keeps its zero weight, so
    everything but its gradient stays finite."""
    P = synth.make_bernoulli_problem(300, 800, 0.05, synth.LOGISTIC, seed=4, support=10)
    assert np.diff(P.col_ptr).min() > 0
    X, y = G.Matrix.of(P), torch.as_tensor(P.y, device="cuda")
    lam = 0.3 * G.lambda_max(X, y, P.loss)
    X.val[int(P.col_ptr[at])] = float("nan")
    for sched in ({}, dict(group=8, piece=256)):
        res = G.solve(X, y, G.make_params(P.loss, lam, rule="shotgun", select_size=10, seed=9,
                                          tol=1e-3, max_epochs=60, **sched))
        assert res.status == G.NOT_CONVERGED, sched
        assert math.isnan(res.stats["kkt_max"]) and math.isfinite(res.stats["objective"]), sched
        assert math.isnan(G.check(X, y, P.loss, lam, res.w).kkt)
        assert res.w[at].item() == 0.0
    prm = G.make_params(P.loss, 0.0, rule="shotgun", select_size=10, seed=9, tol=1e-3, max_epochs=60)
    for st in G.solve_path(X, y, prm, [2.0 * lam, lam], B=16).stats:
        assert not st["converged"] and math.isnan(st["kkt_max"]) and math.isfinite(st["objective"])


def test_drift_of_checks_inside_earlier_launches():
    """z_drift is the largest over all checks: a longer run of the same
    iterates has at least the shorter one's.  16 epochs of 1000 windows fill a
    launch, which thus ends between two checks; the longest run ends in a later
    one, where the weights no longer move and nothing drifts."""
    P = synth.make_bernoulli_problem(400, 1000, 0.01, synth.LOGISTIC, seed=5, support=10)
    X, y = G.Matrix.of(P), torch.as_tensor(P.y, device="cuda")
    lam = 0.3 * G.lambda_max(X, y, P.loss)
    drift = [G.solve(X, y, G.make_params(P.loss, lam, rule="cyclic", tol=0.0, max_epochs=e,
                                         check_every=3)).stats["z_drift"] for e in (3, 15, 399)]
    # the FP64 product that the drift is measured from is summed in any order
    assert 0.0 < drift[0] <= drift[1] * (1 + 1e-6)
    assert drift[1] <= drift[2] * (1 + 1e-6)
