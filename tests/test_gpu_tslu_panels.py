"""GPU parity of the TSLU selection and U in 16-column panels: widths around
the panel edges on short and ragged domains, exact ties, zero columns, rows of
NaN.  Tolerances and checks are test_gpu_tslu's; where every operation is exact
(signed powers of two, one to a row) the results are compared exactly."""
import numpy as np
import pytest

import oracle
import synth
from test_gpu_tslu import check_tslu, dev, host, tl  # noqa: F401

pytestmark = pytest.mark.gpu


# rows and row block: domains of several stages with a ragged last stack; of
# one full stack; of just over b rows; a single stack
@pytest.mark.parametrize("b", [1, 2, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64])
@pytest.mark.parametrize("m,mb", [(2500, 700), (1024, 256), (330, 66), (65, 128), (16384, 4096), (16385, 4096)])
def test_selection_panel_edges(tl, m, mb, b):  # noqa: F811
    print(f"case tslu m={m} b={b} mb={mb}", flush=True)
    check_tslu(tl, synth.gaussian(m, b, seed=1000 * b + m), tl.opts(row_block=mb, tree=2), 2)


@pytest.mark.parametrize("b,zero", [(5, None), (16, 3), (33, 16), (64, 40)])
def test_exact_ties(tl, b, zero):  # noqa: F811
    """Row i holds +-2^(i % 3) in one column: every column's largest entries
    tie exactly, every later stage and level ties again, and a zero column
    leaves only ties of zeros."""
    m, mb = 1500, 400
    i = np.arange(m)
    A = np.zeros((m, b))
    A[i, (7 * i) % b] = np.where(i % 2, -1.0, 1.0) * 2.0 ** (i % 3)
    if zero is not None:
        A[:, zero] = 0.0
    print(f"case ties b={b} zero={zero}", flush=True)
    o = tl.opts(row_block=mb, tree=2)
    ipiv, L, U, info = tl.tslu(dev(A), o)
    ipo, Lo, Uo, info_o = oracle.tslu(A, tl.partition(m, b, o), first=256, stage=256 - b, tree=2)
    assert host(ipiv).tolist() == ipo.tolist() and int(info.item()) == info_o
    assert np.array_equal(host(U), Uo) and np.array_equal(host(L), Lo)


@pytest.mark.parametrize("b", [3, 20, 64])
def test_nan_rows_rank_below_numbers(tl, b):  # noqa: F811
    m = 900
    A = synth.gaussian(m, b, seed=b)
    bad = [0, 255, 256, 600]
    A[bad[:3], :] = np.nan
    A[bad[3], b // 2:] = np.nan
    A[bad[3], : b // 2] = 0.0   # never the largest before its NaN entries
    print(f"case nan rows b={b}", flush=True)
    o = tl.opts(row_block=300, tree=2)
    ipiv, L, U, info = tl.tslu(dev(A), o)
    ipo, Lo, Uo, info_o = oracle.tslu(A, tl.partition(m, b, o), first=256, stage=256 - b, tree=2)
    assert host(ipiv).tolist() == ipo.tolist() and int(info.item()) == info_o
    assert not set(bad) & set(ipo.tolist())
    su = np.abs(Uo).max(axis=0)
    assert np.all(np.abs(host(U) - Uo) <= 1e-13 * su[None, :])
    good = np.setdiff1d(np.arange(m), bad)
    assert np.max(np.abs(host(L) - Lo)[good]) <= 1e-12 * max(1.0, np.abs(Lo[good]).max())
