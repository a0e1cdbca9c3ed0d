"""GPU parity of CALU's trailing update at the edges of its 64 x 64 tiles: one
row or column past a tile, a last panel of one column, tall panels, a padded
leading dimension.  P A = L U within Gaussian elimination's rounding bound
n u |L| |U|, and nothing is written past the rows."""
import numpy as np
import pytest
import torch

import synth
from test_gpu_calu import tl  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n", [(65, 65), (128, 65), (129, 128), (129, 129), (193, 130), (700, 127), (1000, 200),
                                 (257, 257)])
def test_update_edges(tl, m, n):  # noqa: F811
    print(f"case calu m={m} n={n}", flush=True)
    A = synth.gaussian(m, n, seed=3 * m + n)
    a = torch.full((n, m + 5), -7.25, dtype=torch.float64, device="cuda")   # ld m + 5
    a[:, :m] = torch.as_tensor(A.T.copy())
    out = tl.calu(a.t()[:m], tl.opts(row_block=256))
    torch.cuda.synchronize()
    assert bool((a[:, m:] == -7.25).all())   # nothing past the rows is written
    ipiv, info = out[0].cpu().numpy(), int(out[1].item())
    G = a[:, :m].t().cpu().numpy()
    assert info == 0
    P = A.copy()
    for i, p in enumerate(ipiv):
        P[[i, p]] = P[[p, i]]
    L = np.tril(G, -1) + np.eye(m, n)
    U = np.triu(G[:n])
    # n steps of rounding at the size of |L| |U|
    assert np.linalg.norm(P - L @ U) <= n * 2.0 ** -53 * np.linalg.norm(np.abs(L) @ np.abs(U))
