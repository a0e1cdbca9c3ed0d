"""GPU parity of the Cholesky panels at their edges: orders around the 16-row
tiles of the diagonal block and of the rows below it, a failed pivot in each
16-column panel of a block.  Tolerances are test_gpu_chol's."""
import numpy as np
import pytest

import oracle
import synth
from test_gpu_chol import run, tl, tol  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 15, 16, 17, 31, 32, 33, 47, 48, 49, 79, 80, 81, 95, 127, 128, 129, 191, 193, 319,
                               321, 337])
def test_panel_edges(tl, n):  # noqa: F811
    A = synth.spd_gram(n, seed=900 + n)
    Au = A.copy(order="F")
    Au[np.triu_indices(n, 1)] = np.nan   # never read, never written
    G, info = run(tl, Au, n + n % 3)
    Lo, info_o = oracle.cholesky(A)
    assert info == 0 and info_o == 0
    assert np.all(np.isnan(G[np.triu_indices(n, 1)]))
    assert float(np.max(np.abs(np.tril(G) - Lo))) <= tol(n, Lo)


@pytest.mark.parametrize("j", [0, 15, 16, 40, 63, 64, 95, 130])
@pytest.mark.parametrize("bad", [0.0, np.nan])
def test_failed_pivot_in_each_panel(tl, j, bad):  # noqa: F811
    n = 140
    A = synth.spd_gram(n, seed=70 + j)
    A[j, :] = A[:, j] = 0.0
    A[j, j] = bad
    G, info = run(tl, A)
    assert info == j + 1
    done = (j // 64) * 64
    if done:
        Lo, _ = oracle.cholesky(A)
        assert float(np.max(np.abs(np.tril(G)[:, :done] - Lo[:, :done]))) <= tol(n, Lo[:, :done])
