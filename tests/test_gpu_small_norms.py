"""QR of very small matrices: a power of two scales every step exactly as long
as squared norms stay normal numbers, so R of 2^-e A is 2^-e R of A up to the
rounding of the squares that turn denormal (4,096 rows of N(0, 1) entries times
2^-505: squared norms about 2^-998, each square off by at most 2^-1075, their
sum by 2^-1063 or 2^-65 of it).  Allowed: 1e-13 of R's largest entry, test_gpu_parity's
1e-12 for ||Q^T Q - I||."""
import numpy as np
import pytest

import synth
from test_gpu_parity import dev, host, tl  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 5, 16, 40, 64])
@pytest.mark.parametrize("e", [400, 485, 505])
def test_r_scales_with_a(tl, n, e):  # noqa: F811
    m = 4096
    A = synth.gaussian(m, n, seed=n)
    print(f"case {m} x {n} times 2^-{e}", flush=True)
    R = host(tl.factor(dev(A), row_block=512).R())
    f = tl.factor(dev(np.ldexp(A, -e)), row_block=512)
    Rs, Q = np.ldexp(host(f.R()), e), host(f.form_q())
    assert np.max(np.abs(Rs - R)) <= 1e-13 * np.max(np.abs(R))
    assert np.linalg.norm(Q.T @ Q - np.eye(n)) <= 1e-12
