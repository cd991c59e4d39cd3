"""Colouring rounds on the resident grid: equal to the sequential greedy."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_1206_6409_amd import gencd as G
from paper_1206_6409_amd import synth

pytestmark = pytest.mark.gpu


def _check(P):
    want, nc, _ = O.color(P.n, P.k, P.col_ptr, P.row_idx)
    X = G.Matrix.of(P)
    for _ in range(2):  # the second call reuses nothing of the first
        got, n = G.color(X)
        assert n == nc and np.array_equal(got.cpu().numpy(), want)


def _problem(n, k, rows, cols):
    key = np.unique(np.asarray(cols, np.int64) * n + np.asarray(rows, np.int64))
    col_ptr, row_idx, val = synth.coo_to_csc(n, k, key % n, key // n, np.ones(key.size))
    return synth.Problem(n, k, col_ptr, row_idx, val, np.ones(n, np.float32), 0)


# text-like columns (chains of heavy ones), rows longer than two walks of 16
# lanes, columns of one chunk, one more than a chunk and many chunks
@pytest.mark.parametrize("make", [
    lambda: synth.c3_zipf_lasso(scale=0.02),
    lambda: synth.c2_zipf_logistic(scale=0.03),
    lambda: synth.make_bernoulli_problem(300, 900, 0.2, 0, seed=1),
    lambda: synth.make_bernoulli_problem(64, 500, 0.9, 0, seed=2),
    lambda: synth.make_bernoulli_problem(65, 300, 1 - 1e-9, 0, seed=3),
    lambda: synth.make_bernoulli_problem(5000, 40, 0.3, 0, seed=4),
    lambda: synth.make_bernoulli_problem(40000, 9000, 0.0001, 0, seed=5),
    lambda: synth.orthogonal_design(3000, 1000, 0, 6),
])
def test_equal_to_the_sequential_greedy(make):
    _check(make())


def test_more_cut_columns_than_a_round_holds():
    """2000 disjoint columns of 70 entries: one round, 1536 of them cut."""
    cols = np.repeat(np.arange(2000), 70)
    _check(_problem(140000, 2000, np.arange(140000), cols))


def test_more_colours_than_the_grid_holds():
    """A row of 9000 columns: 9000 colours and rounds, over several launches,
    the last ones on the separate kernels."""
    rng = np.random.default_rng(0)
    rows = np.concatenate([np.zeros(9000, np.int64), rng.integers(1, 400, 5000)])
    cols = np.concatenate([np.arange(9000), rng.integers(0, 9000, 5000)])
    _check(_problem(400, 9050, rows, cols))
