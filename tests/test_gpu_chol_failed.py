"""What Cholesky leaves behind a failed pivot is the same on every run.

The trailing update that factors the next diagonal block also tells the other
kernels that a pivot failed; its own tiles finish that update whatever they see
of the word.  With pivot j failing in the diagonal block at t0 = 64 (j / 64):
columns before t0 are L's, the block at t0 and the columns of later 256-column
blocks keep the updates of the block columns before, and the columns of the
update that holds the block (to the end of its 256-column block, or all of them
if t0 starts one) have that update applied.  The tolerance is test_gpu_chol's: the
leading minors before column j are as well conditioned as its matrices.
"""
import numpy as np
import pytest

import synth
from test_gpu_chol import run, tl, tol  # noqa: F401

pytestmark = pytest.mark.gpu


def partial(A, j):
    """The lower triangle the library promises for a failure at column j (64-bit NumPy)."""
    n = A.shape[0]
    W = np.tril(A).astype(np.float64)
    t0 = (j // 64) * 64
    for J in range(0, n, 256):
        jend = min(J + 256, n)
        for s in range(J, jend, 64):
            if s == t0:
                return W
            D = W[s:s + 64, s:s + 64]
            L11 = np.linalg.cholesky(np.tril(D) + np.tril(D, -1).T)
            W[s:s + 64, s:s + 64] = L11
            W[s + 64:, s:s + 64] = np.linalg.solve(L11, W[s + 64:, s:s + 64].T).T
            e = s + 64
            if e < jend:
                k0, cend = s, jend
            elif jend < n:
                k0, cend = J, n
            else:
                continue
            upd = np.tril((W[e:, k0:e] @ W[e:cend, k0:e].T), 0)
            if e == t0:
                b = min(64, n - e)
                upd[:b, :b] = 0.0       # the block that fails is not written
            W[e:, e:cend] -= upd
    return W


@pytest.mark.parametrize("n,j", [(1100, 0), (1100, 70), (1100, 130), (1100, 255), (1100, 256), (1100, 300), (1100, 577),
                                 (1100, 1030), (1100, 1099), (2500, 64), (2500, 300), (2500, 1281)])
def test_partial_factor_is_the_same_on_every_run(tl, n, j):  # noqa: F811
    A = synth.spd_gram(n, seed=31 * n + j)
    A[j, j] = -1.0 - abs(A[j, j])
    print(f"case cholesky n={n} failing at column {j}", flush=True)
    ref = np.tril(partial(A, j))
    first = None
    for _ in range(6):
        G, info = run(tl, A)
        assert info == j + 1
        G = np.tril(G)
        assert float(np.max(np.abs(G - ref))) <= tol(n, ref)
        first = G if first is None else first
        assert np.array_equal(G, first)
