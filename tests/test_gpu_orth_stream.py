"""GPU parity of block orthogonalisation's streaming projections: widths of V
and W around the 16-column tiles and the form's limits (128 and 32 columns),
few rows, a last tile of one row, padded leading dimensions.  Tolerances are
test_gpu_orth's."""
import numpy as np
import pytest
import torch

import oracle
import synth
from test_gpu_orth import colwise, dev, host, tl  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("b", [1, 15, 16, 17, 32, 33])
@pytest.mark.parametrize("m,nv", [(900, 1), (1601, 15), (2049, 16), (3001, 17), (4097, 33), (5000, 64), (6017, 65),
                                  (9000, 97), (20001, 112), (20002, 128), (12000, 129)])
def test_projection_edges(tl, m, nv, b):  # noqa: F811
    print(f"case m={m} nv={nv} b={b}", flush=True)
    rng = np.random.default_rng(m + nv + b)
    V = np.linalg.qr(rng.standard_normal((m, nv)))[0]
    W = synth.gaussian(m, b, seed=nv + b)
    Qo, Ho, Ro = oracle.block_orth(np.asfortranarray(V), W, 1024)
    Vp = torch.full((nv, m + 3), float("nan"), dtype=torch.float64, device="cuda")   # ld m + 3
    Vp[:, :m] = torch.as_tensor(V.T.copy())
    Q, H, R = tl.block_orth(Vp.t()[:m], dev(W), tl.opts(row_block=1024))
    torch.cuda.synchronize()
    Q, H, R = host(Q), host(H), host(R)
    wn = np.linalg.norm(W, axis=0)
    colwise(Q, Qo, 1e-12, np.ones(b))
    colwise(R, Ro, 1e-12, wn)
    colwise(H, Ho, 1e-12, wn)
    B = np.hstack([V, Q])
    assert np.linalg.norm(B.T @ B - np.eye(nv + b)) <= 1e-13
    assert np.linalg.norm(V @ H + Q @ R - W) <= 1e-13 * np.linalg.norm(W)
