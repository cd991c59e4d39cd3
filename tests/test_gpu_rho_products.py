"""Power iteration with the row vector in LDS, at the edges of its row blocks,
lane groups and column chunks, against the FP64 oracle (the same iteration in
another summation order: 1e-10 relative, as in test_gpu_rho)."""
import numpy as np
import pytest

import oracle as O
from paper_1206_6409_amd import gencd as G
from paper_1206_6409_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,k,density", [
    (700, 9000, 0.02),       # one block, 14 entries a column
    (3000, 2500, 0.02),      # 60 entries
    (19456, 400, 0.02),      # exactly one block
    (19457, 400, 0.02),      # two blocks of unequal size
    (38912, 300, 0.02),      # two full blocks
    (38913, 300, 0.01),      # three
    (58368, 200, 0.02),      # three full blocks
    (58369, 200, 0.02),      # beyond: global atomics
    (300, 40000, 0.02),      # 6 entries, many columns per chunk
])
def test_rho_matches_the_oracle(n, k, density):
    P = synth.make_bernoulli_problem(n, k, density, synth.SQUARED, seed=n + k, support=10)
    _, want, live = O.rho(O.Matrix.of(P), 6)
    got = G.estimate_rho(G.Matrix.of(P), 6)
    assert got.k_live == live
    np.testing.assert_allclose(got.history, want, rtol=1e-10)


def test_heavy_column_and_empty_columns():
    """A dense column spans several chunks; empty columns get no product."""
    P = synth.make_bernoulli_problem(20000, 600, 0.01, synth.SQUARED, seed=3, support=10)
    rng = np.random.default_rng(1)
    rows = np.arange(20000, dtype=np.int32)
    cut = int(P.col_ptr[300])
    col_ptr = np.concatenate([P.col_ptr[:301], P.col_ptr[300:] + 20000, [P.col_ptr[-1] + 20000] * 5])
    Q = synth.Problem(P.n, col_ptr.size - 1, col_ptr,
                      np.concatenate([P.row_idx[:cut], rows, P.row_idx[cut:]]),
                      np.concatenate([P.val[:cut], rng.standard_normal(20000).astype(np.float32),
                                      P.val[cut:]]), P.y, P.loss)
    _, want, _ = O.rho(O.Matrix.of(Q), 8)
    np.testing.assert_allclose(G.estimate_rho(G.Matrix.of(Q), 8).history, want, rtol=1e-10)
