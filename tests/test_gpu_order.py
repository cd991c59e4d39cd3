"""The epoch order (permutation, window bounds, long columns' pieces) through
the solves that use it, against the oracle's iterates.  After an epoch or two
the weights differ by FP32 rounding only: a column's tree-summed gradient is
off by a few ulps of sum |x r|, about two decimal digits above its own size
where terms cancel, so 1e-5 (170 ulps) in the 2-norm."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_1206_6409_amd import gencd as G
from paper_1206_6409_amd import synth

pytestmark = pytest.mark.gpu
RULES = {"cyclic": O.CYCLIC, "shotgun": O.SHOTGUN, "greedy": O.GREEDY}


def _rel(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


def _check(P, rule, S, epochs, ratio, **kw):
    Xo = O.Matrix.of(P)
    lam = ratio * O.lambda_max(Xo, P.y, P.loss)
    ref = O.solve(Xo, P.y, P.loss, lam, RULES[rule], select_size=S, seed=5, tol=0.0,
                  max_epochs=epochs, check_every=epochs)
    assert np.linalg.norm(ref.w) > 0
    prm = G.make_params(P.loss, lam, rule=rule, select_size=S, seed=5, tol=0.0, max_epochs=epochs,
                        check_every=epochs, **kw)
    res = G.solve(G.Matrix.of(P), torch.as_tensor(P.y, device="cuda"), prm)
    assert res.stats["iters"] == ref.iters
    assert _rel(res.w.cpu().numpy().astype(np.float64), ref.w) <= 1e-5


# one position, edges of a tile of 1024 positions, several tiles, windows that
# end with a tile, inside it and past it; `piece` 64 with columns of 120 entries splits them
@pytest.mark.parametrize("k,rule,S,piece", [
    (1, "shotgun", 1, 256), (1023, "shotgun", 100, 256), (1024, "shotgun", 256, 64),
    (1025, "shotgun", 256, 64), (2048, "shotgun", 1024, 256), (2049, "shotgun", 300, 64),
    (5000, "shotgun", 37, 256), (1025, "cyclic", 1, 64), (1025, "greedy", 0, 256),
    (3001, "greedy", 0, 64),
])
def test_order_of_a_solve(k, rule, S, piece):
    P = synth.make_bernoulli_problem(400, k, 0.05 if piece > 64 else 0.3, synth.LOGISTIC, 11,
                                     support=min(20, k))
    _check(P, rule, S, 2, 0.5, group=8, piece=piece)


def test_order_past_the_table():
    """More live columns than the one-launch order takes."""
    n, k = 1 << 16, (1 << 22) + 5
    rng = np.random.default_rng(0)
    P = synth.Problem(n=n, k=k, col_ptr=np.arange(k + 1, dtype=np.int64),
                      row_idx=rng.integers(0, n, k).astype(np.int32),
                      val=rng.standard_normal(k).astype(np.float32),
                      y=np.where(rng.random(n) < 0.5, 1.0, -1.0).astype(np.float32),
                      loss=synth.LOGISTIC, w_true=np.zeros(k), name="singles")
    _check(P, "shotgun", 1 << 20, 1, 0.9)
