"""Windows of more work units than the resident grid has waves: the units past
the registers, split columns among them.  Against the separate launches of
GENCD_PROFILE; after two epochs the weights differ by FP32 rounding only (a few
ulps of a gradient's sums, about two decimal digits above its own size where
terms cancel: 1e-5 in the 2-norm)."""
import numpy as np
import pytest
import torch

from paper_1206_6409_amd import gencd as G
from paper_1206_6409_amd import synth

pytestmark = pytest.mark.gpu

WAVES = 1024  # of the larger grid, 64 workgroups


def _units(P, S, group, piece):
    """Expected units of a window: 64 / group columns, or one piece of a long one."""
    ln = np.diff(P.col_ptr)
    ln = ln[ln > 0]
    pieces = np.ceil(ln[ln > 4 * group] / piece).sum()
    return -(-S * group // 64) + S * pieces / ln.size


def _kernels(fn):
    from torch.profiler import ProfilerActivity, profile
    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        fn()
        torch.cuda.synchronize()
    return {e.name for e in prof.events()}


def _rel(a, b):
    return float((a.double() - b.double()).norm() / b.double().norm())


def _compare(P, kernel, lam_ratio=0.05, **kw):
    X, y = G.Matrix.of(P), torch.as_tensor(P.y, device="cuda")
    lam = lam_ratio * G.lambda_max(X, y, P.loss)
    kw = dict(seed=3, tol=0.0, max_epochs=2, **kw)
    out = []
    names = _kernels(lambda: out.append(G.solve(X, y, G.make_params(P.loss, lam, **kw))))
    assert any(kernel in s for s in names)
    want = G.solve(X, y, G.make_params(P.loss, lam, **dict(kw, flags=G.PROFILE)))
    for key in ("iters", "coord_updates", "nnz_updates"):
        assert out[0].stats[key] == want.stats[key], key
    assert _rel(out[0].w, want.w) <= 1e-5 and _rel(out[0].z, want.z) <= 1e-5


@pytest.mark.parametrize("S,group,piece,flags", [
    (4090, 16, 128, 0),            # short columns and pieces past the registers
    (2040, 32, 64, G.USE_GRAPH),   # many pieces of a split column
    (4300, 4, 64, 0),              # mostly pieces
])
def test_accept_all_windows(S, group, piece, flags):
    P = synth.c2_zipf_logistic(scale=0.05)
    assert _units(P, S, group, piece) > WAVES
    _compare(P, "k_epoch_grid", rule="shotgun", select_size=S, group=group, piece=piece,
             residual=1, flags=flags)


@pytest.mark.parametrize("S,B,mean,group", [
    (10_000, 256, 1.5, 8),   # short columns, the largest blocks
    (600, 100, 40, 32),      # blocks of two rounds of a wave
    (400, 2, 60, 8),         # long columns, a block each for half the positions
])
def test_thread_greedy_windows(S, B, mean, group):
    P = synth.make_bernoulli_problem(60_000, 8 * S, mean / 60_000, synth.LOGISTIC, seed=S, support=50)
    if S == 10_000:
        assert _units(P, S, group, 256) > WAVES
    assert S * P.nnz / (np.diff(P.col_ptr) > 0).sum() <= 32768
    _compare(P, "k_greedy_grid", rule="thread_greedy", select_size=S, block=B, group=group,
             piece=256)


@pytest.mark.parametrize("flags", [0, G.USE_GRAPH])
def test_colour_class_larger_than_the_grid(flags):
    """One class of 12000 columns of up to three entries and one of 300, and 60
    classes of one column."""
    rng = np.random.default_rng(5)
    k0, long_len, n = 12_000, 300, 40_000
    lens = np.concatenate([rng.integers(1, 4, k0), [long_len]])
    cols = np.repeat(np.arange(k0 + 1), lens)
    rows = rng.permutation(n)[:cols.size]
    cols = np.concatenate([cols, k0 + 1 + np.repeat(np.arange(60), 40)])
    rows = np.concatenate([rows, np.concatenate([rng.permutation(n)[:40] for _ in range(60)])])
    k = k0 + 61
    col_ptr, row_idx, val = synth.coo_to_csc(n, k, rows, cols, rng.standard_normal(rows.size))
    y = np.where(rng.random(n) < 0.5, 1.0, -1.0).astype(np.float32)
    P = synth.Problem(n, k, col_ptr, row_idx, val, y, synth.LOGISTIC)
    color = np.concatenate([np.zeros(k0 + 1), np.arange(1, 61)]).astype(np.int32)
    assert -(-(k0 + 1) // 8) > WAVES
    _compare(P, "k_epoch_grid", lam_ratio=0.1, rule=G.COLORING, num_colors=61, flags=flags,
             colors=torch.as_tensor(color, device="cuda"))


def test_preset_blocks_of_unequal_windows():
    P = synth.c2_zipf_logistic(scale=0.05)
    _compare(P, "k_epoch_grid", rule=G.BLOCK_SHOTGUN, block=6, residual=1)
