"""TSLU's U and L11 where a chosen row holds an infinity or a NaN, or a pivot
is zero: elimination without pivoting touches the rows below the pivot only,
and none below a zero pivot, whose column of L11 keeps what stands there.  The
reference is that elimination in NumPy on the rows the library chose; entries
that are not finite are compared as they are, finite ones with test_gpu_tslu's
tolerance on U (1e-13 of the column's largest finite entry)."""
import numpy as np
import pytest

import synth
from test_gpu_tslu import dev, host, tl  # noqa: F401

pytestmark = pytest.mark.gpu


def eliminate(P):
    """L11 (unit lower) and U of the rows P in pivot order."""
    M = P.copy()
    b = M.shape[0]
    with np.errstate(all="ignore"):
        for k in range(b):
            if M[k, k] != 0.0:
                M[k + 1:, k] = M[k + 1:, k] / M[k, k]
                M[k + 1:, k + 1:] -= M[k + 1:, k:k + 1] * M[k:k + 1, k + 1:]
    return np.tril(M, -1) + np.eye(b), np.triu(M)


def same(G, ref):
    kind = np.isfinite(ref)
    assert np.array_equal(np.isfinite(G), kind)
    assert np.array_equal(G[~kind], ref[~kind], equal_nan=True)
    scale = np.where(kind, np.abs(np.where(kind, ref, 0.0)), 0.0).max(axis=0)
    assert np.all(np.abs(np.where(kind, G, 0.0) - np.where(kind, ref, 0.0)) <= 1e-13 * np.maximum(scale, 1.0)[None, :])


def check(tl, A, what):  # noqa: F811
    b = A.shape[1]
    print(f"case {what} {A.shape[0]} x {b}", flush=True)
    ipiv, L, U, info = tl.tslu(dev(A), tl.opts(row_block=256, tree=2))
    rows = host(ipiv)
    L11, Uo = eliminate(A[rows])
    same(host(U), Uo)
    same(host(L)[rows], L11)
    zero = np.nonzero(np.diag(Uo) == 0.0)[0]
    assert int(info.item()) == (zero[0] + 1 if len(zero) else 0)
    return rows, Uo


@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
@pytest.mark.parametrize("b,k,j", [(3, 0, 2), (16, 5, 6), (20, 0, 15), (33, 14, 18), (64, 17, 63), (64, 40, 45)])
def test_a_pivot_row_is_not_finite_past_its_pivot(tl, b, k, j, bad):  # noqa: F811
    """Row 7 is pivot k (the largest by far in column k, zero before it)."""
    A = synth.gaussian(600, b, seed=b + k)
    A[7, :k] = 0.0
    A[7, k] = 1e3
    A[7, j] = bad
    rows, U = check(tl, A, f"pivot {k} holds {bad} in column {j}")
    assert rows[k] == 7 and not np.isfinite(U[k, j])
    assert np.all(np.isfinite(U[:k, :]))      # earlier rows of U stay finite


@pytest.mark.parametrize("b,z", [(4, 1), (16, 0), (20, 3), (33, 15), (33, 16), (64, 30)])
def test_zero_pivot_over_nan(tl, b, z):  # noqa: F811
    """b rows in all; column z has zeros and, in the last rows, NaN: its pivot
    is zero and the NaN below it reach no other column of U."""
    A = np.triu(synth.gaussian(b, b, seed=b + z)) + 4.0 * np.eye(b)
    A[:, z] = 0.0
    A[b - 1, z] = np.nan
    rows, U = check(tl, A, f"zero pivot {z} over a NaN")
    assert np.all(np.isfinite(U))
    assert sorted(rows.tolist()) == list(range(b))
