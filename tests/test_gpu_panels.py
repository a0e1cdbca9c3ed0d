"""GPU parity of the 16-column panel QR at its edges: widths around the panel
and slot boundaries, chunks that end in a partial tile, domains of a single
short chunk, columns that cannot be read in 16-byte pieces, and reflectors
that are exactly the identity.  Tolerances and checks are test_gpu_parity's."""
import numpy as np
import pytest

import synth
from test_gpu_parity import check_all, dev, host, rel, tl  # noqa: F401

pytestmark = pytest.mark.gpu


# rows: 3 domains of 512 and a tail of 257 (one full chunk of a wide panel and
# one row; odd, so no 16-byte column starts), the same one row longer (even),
# a single domain of one partial chunk
@pytest.mark.parametrize("n", [1, 7, 8, 9, 15, 16, 17, 24, 31, 32, 33, 47, 48, 49, 63, 64])
@pytest.mark.parametrize("m,mb", [(1793, 512), (1794, 512), (70, 128)])
def test_panel_edges(tl, m, n, mb):  # noqa: F811
    check_all(tl, synth.gaussian(m, n, seed=100 * n + m % 7), mb=mb)


@pytest.mark.parametrize("n,zero", [(16, 0), (33, 20), (64, 63), (64, 16)])
def test_identity_reflectors(tl, n, zero):  # noqa: F811
    """A zero column gives tau = 0 in every chunk and a zero column of R.  R
    is not unique then (the identity leaves its pivot row out of the later
    eliminations), but Q R = A and R^T R = A^T A still hold: with
    ||A - Q R|| <= 1e-13 ||A||, the latter to 2e-13 ||A||_F^2."""
    A = synth.gaussian(1500, n, seed=n + zero)
    A[:, zero] = 0.0
    f = tl.factor(dev(A), row_block=512)
    R, Q = host(f.R()), host(f.form_q())
    assert np.all(R[:, zero] == 0.0)
    assert rel(Q @ R, A) <= 1e-13
    assert np.linalg.norm(R.T @ R - A.T @ A) <= 2e-13 * np.linalg.norm(A) ** 2
