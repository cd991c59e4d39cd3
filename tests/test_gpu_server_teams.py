"""Server rounds on teams of resident workgroups against the oracle's Jacobi
iterates.  After two epochs the weights differ by FP32 rounding only: a
column's tree-summed gradient is off by a few ulps of sum |x r|, about two
decimal digits above its own size where terms cancel, so 1e-5 (170 ulps) in
the 2-norm."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_1206_6409_amd import gencd as G
from paper_1206_6409_amd import synth

pytestmark = pytest.mark.gpu
EPOCHS = 2


def _rel(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


def _bern(n, k, density, loss, seed):
    return synth.make_bernoulli_problem(n, k, density, loss, seed, support=20)


# (problem, |J|, lambda / lambda_max): one window per epoch; single columns, so
# an epoch of many launches; a ragged last window; every lane-group size (mean
# lengths 4 to 300); more units than 64 workgroups have waves; long columns
# (several batches); many small requests at once; windows above the line, on
# two launches, next to small ones
MIXES = {
    "one": [(("bern", 300, 400, 0.02, synth.LOGISTIC), 400, 0.8)],
    "shapes": [
        (("bern", 300, 400, 0.02, synth.LOGISTIC), 1, 0.3),
        (("bern", 400, 1001, 0.01, synth.SQUARED), 50, 0.3),
        (("bern", 1000, 700, 0.02, synth.LOGISTIC), 33, 0.3),
        (("bern", 1500, 600, 0.06, synth.SQUARED), 17, 0.3),
        (("bern", 2000, 500, 0.15, synth.LOGISTIC), 9, 0.3),
        (("zipf", 0.02), 60, 0.3),
    ],
    "units": [(("bern", 400, 20000, 0.01, synth.LOGISTIC), 18000, 0.8)],
    "many": [(("bern", 300, 400, 0.02, synth.LOGISTIC), 5 + i, 0.3) for i in range(40)],
    "large": [(("bern", 4000, 6000, 0.02, synth.LOGISTIC), 4000, 0.8),
              (("bern", 400, 1001, 0.01, synth.SQUARED), 50, 0.3)],
}


@pytest.mark.parametrize("name", list(MIXES))
def test_team_rounds_match_the_oracle(name):
    print("CASE server teams", name, flush=True)
    jobs, need = [], 0
    for i, (what, S, ratio) in enumerate(MIXES[name]):
        P = synth.c2_zipf_logistic(scale=what[1]) if what[0] == "zipf" else _bern(*what[1:], seed=i)
        Xo = O.Matrix.of(P)
        lam = ratio * O.lambda_max(Xo, P.y, P.loss)
        ref = O.solve(Xo, P.y, P.loss, lam, O.SHOTGUN, select_size=S, seed=3, tol=0.0,
                      max_epochs=EPOCHS, check_every=EPOCHS)
        X, y = G.Matrix.of(P), torch.as_tensor(P.y, device="cuda")
        prm = G.make_params(P.loss, lam, rule=G.SHOTGUN, select_size=S, seed=3, tol=0.0,
                            max_epochs=EPOCHS, check_every=EPOCHS)
        need += G.Server.request_bytes(X, prm)
        w = torch.empty(P.k, dtype=torch.float32, device="cuda")
        z = torch.empty(P.n, dtype=torch.float32, device="cuda")
        jobs.append((ref, X, y, prm, w, z))
    srv = G.Server(G.Server.overhead_bytes(len(jobs)) + need + 4096, max_slots=len(jobs))
    torch.cuda.synchronize()
    for _ in range(2):  # the second time into used slots
        for i, (ref, X, y, prm, w, z) in enumerate(jobs):
            srv.submit(X, y, prm, w, z, tag=i)
        left, res = len(jobs), {}
        while left:
            for r in srv.poll(wait_for=1):
                res[r["user_tag"]] = r
                left -= 1
        for i, (ref, X, y, prm, w, z) in enumerate(jobs):
            assert res[i]["stats"]["iters"] == ref.iters, (i, res[i])
            assert np.linalg.norm(ref.w) > 0
            assert _rel(w.cpu().numpy().astype(np.float64), ref.w) <= 1e-5, i
            assert _rel(z.cpu().numpy().astype(np.float64), ref.z) <= 1e-5, i
    info = srv.info()
    srv.close()
    # rounds run on while the last check is read back
    assert info["slot_rounds"] >= 2 * sum(j[0].iters for j in jobs), info
