"""The server does not run far ahead of the results it waits for."""
import pytest
import torch

from paper_1206_6409_amd import gencd as G
from paper_1206_6409_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("slots", [1, 4])
def test_few_windows_run_past_a_request(slots):
    """Requests of one epoch of 400 windows.  Rounds go on until the last check
    has been read back, for at most the windows in flight (64, and a launch of 32
    that was being enqueued) and about as many again before it is looked at; with
    eight launches in flight it was about 250."""
    P = synth.make_bernoulli_problem(4000, 20_000, 20 / 4000, synth.LOGISTIC, seed=1, support=20)
    X, y = G.Matrix.of(P), torch.as_tensor(P.y, device="cuda")
    prm = G.make_params(P.loss, 0.1 * G.lambda_max(X, y, P.loss), rule="shotgun", select_size=50,
                        seed=3, tol=0.0, max_epochs=1)
    srv = G.Server(G.Server.overhead_bytes(slots) + slots * G.Server.request_bytes(X, prm) + 4096,
                   max_slots=slots)
    ws = [torch.empty(P.k, dtype=torch.float32, device="cuda") for _ in range(6)]
    torch.cuda.synchronize()
    iters = 0
    for i, w in enumerate(ws):
        srv.submit(X, y, prm, w, tag=i)
    left = len(ws)
    while left:
        for r in srv.poll(wait_for=1):
            iters += r["stats"]["iters"]
            left -= 1
    info = srv.info()
    srv.close()
    assert iters == len(ws) * 400
    print("windows past the end", (info["slot_rounds"] - iters) / len(ws))
    assert info["slot_rounds"] - iters <= len(ws) * 160
