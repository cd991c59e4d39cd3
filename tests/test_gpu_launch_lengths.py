"""No launch runs an unbounded number of windows: long epochs are cut, and the
cut changes nothing."""
import numpy as np
import pytest
import torch

from paper_1206_6409_amd import gencd as G
from paper_1206_6409_amd import synth

pytestmark = pytest.mark.gpu


def _kernels(fn):
    """Names of the kernels that fn launches."""
    from torch.profiler import ProfilerActivity, profile
    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        fn()
        torch.cuda.synchronize()
    return [e.name for e in prof.events()]


# (rows, rule, |J|, kernel, windows of an epoch, most windows of a launch).
# One workgroup below 13312 rows, the resident grid above.
@pytest.mark.parametrize("n,rule,S,kernel,limit", [
    (300, "cyclic", 1, "k_solo", 16384),
    (14000, "cyclic", 1, "k_epoch_grid", 4096),
    (14000, "thread_greedy", 2, "k_greedy_grid", 4096),
])
def test_long_epochs_are_cut(n, rule, S, kernel, limit):
    P = synth.make_bernoulli_problem(n, 40000, 3.0 / n, synth.LOGISTIC, seed=2, support=10)
    live = int((np.diff(P.col_ptr) > 0).sum())
    windows = -(-live // S)
    X, y = G.Matrix.of(P), torch.as_tensor(P.y, device="cuda")
    lam = 0.1 * G.lambda_max(X, y, P.loss)
    kw = dict(rule=rule, select_size=S, block=2, seed=9, tol=0.0, max_epochs=1)
    out = []
    names = _kernels(lambda: out.append(G.solve(X, y, G.make_params(P.loss, lam, **kw))))
    assert sum(kernel in s for s in names) == -(-windows // limit) > 1
    # the separate launches of GENCD_PROFILE: the same windows, FP32 rounding apart
    want = G.solve(X, y, G.make_params(P.loss, lam, flags=G.PROFILE, **kw))
    assert out[0].stats["iters"] == want.stats["iters"] == windows
    assert out[0].stats["coord_updates"] == want.stats["coord_updates"]
    a, b = out[0].w.double(), want.w.double()
    # columns of a few entries: a few ulps of their gradients' sums
    assert float((a - b).norm() / b.norm()) <= 1e-5
