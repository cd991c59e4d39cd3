"""Epochs on the grid of resident workgroups against the oracle's Jacobi
iterates.  After two epochs the weights differ by FP32 rounding only: a column's
tree-summed gradient is off by a few ulps of sum |x r|, about two decimal
digits above its own size where terms cancel, so 1e-5 (170 ulps) in the
2-norm."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_1206_6409_amd import gencd as G
from paper_1206_6409_amd import synth

pytestmark = pytest.mark.gpu


def _rel(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


# windows that leave most waves idle, more work units than waves (long pieces
# and short columns), single columns, a nearly empty last window, split columns
# of many pieces, every lane-group size, the largest piece
@pytest.mark.parametrize("scale,S,group,piece,flags", [
    (0.05, 100, 8, 256, 0),
    (0.05, 1, 8, 256, 0),
    (0.05, 1024, 4, 64, 0),
    (0.05, 4097, 16, 128, 0),
    (0.05, 4000, 32, 256, 0),
    (0.05, 333, 8, 64, G.USE_GRAPH),
    (0.2, 8000, 4, 64, 0),
    (0.2, 700, 8, 256, G.USE_GRAPH),
])
def test_windows_match_the_oracle(scale, S, group, piece, flags):
    P = synth.c2_zipf_logistic(scale=scale)
    Xo = O.Matrix.of(P)
    lam = 0.05 * O.lambda_max(Xo, P.y, P.loss)
    epochs = 1 if S == 1 else 2
    ref = O.solve(Xo, P.y, P.loss, lam, O.SHOTGUN, select_size=S, seed=3, tol=0.0,
                  max_epochs=epochs)
    X, y = G.Matrix.of(P), torch.as_tensor(P.y, device="cuda")
    prm = G.make_params(P.loss, lam, rule=G.SHOTGUN, select_size=S, seed=3, tol=0.0,
                        max_epochs=epochs, group=group, piece=piece, flags=flags)
    for _ in range(2):  # a second solve on the same workspace, with eager work between
        res = G.solve(X, y, prm)
        torch.cuda.synchronize()
        assert res.stats["iters"] == ref.iters
        assert _rel(res.w.cpu().numpy().astype(np.float64), ref.w) <= 1e-5
        assert _rel(res.z.cpu().numpy().astype(np.float64), ref.z) <= 1e-5


@pytest.mark.parametrize("flags", [0, G.USE_GRAPH])
def test_coloring_matches_the_oracle(flags):
    """Colour classes as windows, one of them empty."""
    P = synth.c3_zipf_lasso(scale=0.02)
    Xo = O.Matrix.of(P)
    lam = 0.1 * O.lambda_max(Xo, P.y, P.loss)
    col, nc, _ = O.color(P.n, P.k, P.col_ptr, P.row_idx)
    col = np.where(col >= 5, col + 1, col).astype(np.int32)  # colour 5 has no columns
    ref = O.solve(Xo, P.y, P.loss, lam, O.COLORING, colors=col, seed=3, tol=0.0, max_epochs=2)
    X, y = G.Matrix.of(P), torch.as_tensor(P.y, device="cuda")
    res = G.solve(X, y, G.make_params(P.loss, lam, rule=G.COLORING, seed=3, tol=0.0, max_epochs=2,
                                      colors=torch.as_tensor(col, device="cuda"),
                                      num_colors=nc + 1, flags=flags))
    assert _rel(res.w.cpu().numpy().astype(np.float64), ref.w) <= 1e-5


def test_concurrent_solves_on_two_streams():
    """Two grids at once on one device: each enrols its own workgroups."""
    P = synth.c2_zipf_logistic(scale=0.05)
    X, y = G.Matrix.of(P), torch.as_tensor(P.y, device="cuda")
    lam = 0.05 * G.lambda_max(X, y, P.loss)
    prm = [G.make_params(P.loss, lam, rule=G.SHOTGUN, select_size=500, seed=s, tol=0.0,
                         max_epochs=20, check_every=20, group=8, piece=256) for s in (1, 2)]
    want = [G.solve(X, y, p).w.cpu().numpy() for p in prm]
    import threading
    got = [None, None]

    def work(i):
        st = torch.cuda.Stream()
        with torch.cuda.stream(st):
            got[i] = G.solve(X, y, prm[i]).w.cpu().numpy()

    torch.cuda.synchronize()
    ts = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    for i in range(2):
        assert _rel(got[i].astype(np.float64), want[i].astype(np.float64)) <= 1e-5


# blocks of one to several rounds of a wave, ragged last blocks and windows,
# winners that one wave scatters and winners spread over the grid (columns of
# more than 1024 entries win their blocks), graph replays
@pytest.mark.parametrize("scale,S,B,group,piece,flags", [
    (0.05, 1024, 64, 8, 256, 0),
    (0.05, 1000, 100, 4, 64, G.USE_GRAPH),
    (0.05, 333, 2, 16, 128, 0),
    (0.05, 4097, 256, 32, 256, 0),
    (0.2, 512, 32, 8, 256, G.USE_GRAPH),
])
def test_thread_greedy_matches_the_separate_launches(scale, S, B, group, piece, flags):
    """GENCD_PROFILE keeps one launch per phase; the picks of two epochs are
    the same and the weights differ by FP32 rounding."""
    P = synth.c2_zipf_logistic(scale=scale)
    X, y = G.Matrix.of(P), torch.as_tensor(P.y, device="cuda")
    lam = 0.05 * G.lambda_max(X, y, P.loss)
    kw = dict(rule=G.THREAD_GREEDY, select_size=S, block=B, seed=3, tol=0.0, max_epochs=2,
              group=group, piece=piece)
    a = G.solve(X, y, G.make_params(P.loss, lam, flags=flags, **kw))
    b = G.solve(X, y, G.make_params(P.loss, lam, flags=G.PROFILE, **kw))
    for key in ("iters", "coord_updates", "nnz_updates"):
        assert a.stats[key] == b.stats[key], key
    assert _rel(a.w.cpu().numpy().astype(np.float64), b.w.cpu().numpy().astype(np.float64)) <= 1e-5
    assert _rel(a.z.cpu().numpy().astype(np.float64), b.z.cpu().numpy().astype(np.float64)) <= 1e-5
