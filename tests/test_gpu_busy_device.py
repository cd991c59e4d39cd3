"""Resident grids on a device that other work keeps busy: the results are those
of an idle device."""
import threading
import time

import numpy as np
import pytest
import torch

import oracle as O
from paper_1206_6409_amd import gencd as G
from paper_1206_6409_amd import synth

pytestmark = pytest.mark.gpu


class Busy:
    """Long rows summed on a stream of their own, a few kernels ahead: most
    compute units hold long-running workgroups of it."""

    def __init__(self, rows):
        self.a = torch.rand(rows, 400_000, device="cuda")
        self.b = torch.empty_like(self.a)
        self.stop = False
        self.thread = threading.Thread(target=self.work)

    def work(self):
        with torch.cuda.stream(torch.cuda.Stream()):
            ahead = []
            while not self.stop:
                torch.cumsum(self.a, 1, out=self.b)
                ahead.append(torch.cuda.Event())
                ahead[-1].record()
                if len(ahead) > 4:
                    ahead.pop(0).synchronize()
            torch.cuda.current_stream().synchronize()

    def __enter__(self):
        self.thread.start()
        time.sleep(0.1)

    def __exit__(self, *exc):
        self.stop = True
        self.thread.join()


def _rel(a, b):
    return float((a.double() - b.double()).norm() / b.double().norm())


# one epoch of Thread-Greedy: proxies that agree to FP32 rounding may swap picks
@pytest.mark.parametrize("rule,S,epochs,flags", [
    ("shotgun", 5000, 20, 0), ("shotgun", 5000, 20, G.USE_GRAPH), ("shotgun", 200, 4, 0),
    ("thread_greedy", 1000, 1, 0)])
def test_results_beside_other_work(rule, S, epochs, flags):
    """1600 rows: six workgroups of 256 on every compute unit, which leave the
    grid's workgroups of 1024 threads little room, so that fewer than asked for
    enrol."""
    P = synth.make_bernoulli_problem(100_000, 100_000, 1e-4, synth.LOGISTIC, seed=1, support=50)
    X, y = G.Matrix.of(P), torch.as_tensor(P.y, device="cuda")
    lam = 0.1 * G.lambda_max(X, y, P.loss)

    def solve():
        prm = G.make_params(P.loss, lam, rule=rule, select_size=S, block=32, seed=3, tol=0.0,
                            max_epochs=epochs, check_every=2, flags=flags)
        return G.solve(X, y, prm, ws=ws)

    ws = G.workspace(X, G.make_params(P.loss, lam, rule=rule, select_size=S, block=32))
    want = solve()
    with Busy(1600):
        runs = [solve() for _ in range(3)]
    for res in runs:
        for key in ("epochs", "iters", "coord_updates", "nnz_visits", "nnz_updates"):
            assert res.stats[key] == want.stats[key], key
        # the same windows; FP32 sums in another order
        assert _rel(res.w, want.w) <= 1e-5 and _rel(res.z, want.z) <= 1e-5


def test_colouring_beside_other_work():
    P = synth.c3_zipf_lasso(scale=0.02)
    want, nc, _ = O.color(P.n, P.k, P.col_ptr, P.row_idx)
    with Busy(1600):
        got, n = G.color(G.Matrix.of(P))
        assert n == nc and np.array_equal(got.cpu().numpy(), want)
