"""The chained apply where it walks: 256 domains and more, so that a workgroup
takes blocks of 32 columns, a second item and padding items (the domains are not
a multiple of 8), in domains of one short chunk, of two chunks and a rest, of
under and over 256 rows; Q^T and Q against the oracle with test_gpu_parity's
tolerances.  A mixed factor of two panels does the same to its trailing columns:
its solve meets test_gpu_mixed's backward error.

Its rounding: B - V Z rounds once at B's size whether there are 16 columns (the
three-pass form) or more (the chained one), so ||B - Q Q^T B|| / ||B|| of the two
agree; norms over 2e6 rounding errors spread by less than a percent, the orders
of the sums in W and Z differ, and 1.15 is allowed.  Summing V Z into B, one
rounding per four columns of V, makes it 1.37."""
import numpy as np
import pytest
import torch

import oracle
import synth
from test_gpu_mixed import eta
from test_gpu_parity import colwise, dev, host, rel, tl  # noqa: F401

pytestmark = pytest.mark.gpu


# 263 domains of 64 (520) rows, the last with the rest or, where the rest has n rows, a 264th
@pytest.mark.parametrize("mb,extra,n,k", [(64, 17, n, k) for n in (8, 24, 40, 64) for k in (17, 31, 33, 50)] +
                         [(520, 9, n, k) for n in (8, 16, 40, 64) for k in (17, 50)] +
                         [(256, 5, 8, 33), (250, 7, 16, 33)])
def test_long_walks(tl, mb, extra, n, k):  # noqa: F811
    m = 263 * mb + extra
    print(f"case m={m} n={n} k={k} mb={mb}", flush=True)
    A, B = synth.gaussian(m, n, seed=n + k), synth.gaussian(m, k, seed=n + 7 * k)
    orc = oracle.TSQR(A, mb=mb, tree=2)
    f = tl.factor(dev(A), row_block=mb, tree=2)
    Bd = dev(B)
    f.apply_qt_(Bd)
    C, Co = host(Bd), orc.apply_qt(B)
    assert rel(C[:n], Co[:n]) <= 1e-12
    colwise(C[:n], Co[:n], 1e-12, scale=np.linalg.norm(B, axis=0))
    assert np.allclose(np.linalg.norm(C[n:], axis=0), np.linalg.norm(Co[n:], axis=0), rtol=1e-11,
                       atol=1e-13 * np.linalg.norm(B))
    f.apply_q_(Bd)
    assert rel(host(Bd), B) <= 1e-13


@pytest.mark.parametrize("n", [100, 128])
def test_mixed_trailing_columns(tl, n):  # noqa: F811
    m, mb = 263 * 128 + 17, 128
    print(f"case mixed m={m} n={n} mb={mb}", flush=True)
    A, b = synth.gaussian(m, n, seed=n), synth.gaussian(m, 1, seed=n + 1)
    f = tl.factor(dev(A), prec=tl.MIXED, row_block=mb)
    X, _, info = f.lsq(dev(b), A=dev(A))
    assert int(info.item()) == 0 and eta(A, host(X)[:, 0], b[:, 0]) <= 1e-12


def test_rounds_like_the_form_for_few_columns(tl):  # noqa: F811
    m, n = 131072, 128
    g = torch.Generator(device="cuda").manual_seed(1)
    f = tl.factor(torch.randn((n, m), generator=g, device="cuda", dtype=torch.float64).t(), row_block=4096)
    err = []
    for k in (16, 17):
        B0 = torch.randn((k, m), generator=g, device="cuda", dtype=torch.float64).t()
        B = B0.t().clone().t()
        f.apply_qt_(B)
        f.apply_q_(B)
        err.append(float((B - B0).norm() / B0.norm()))
        print(f"case {m} x {n}, {k} columns: ||B - Q Q^T B|| / ||B|| {err[-1]:.2e}", flush=True)
    assert err[1] <= 1.15 * err[0]
