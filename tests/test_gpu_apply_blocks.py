"""GPU parity of applying Q^T and Q to blocks of columns: widths around the
16-row tiles and the 16-column blocks, every tree shape (a chain of several
rights per node among them), short last domains.  Tolerances are
test_gpu_parity's."""
import numpy as np
import pytest

import oracle
import synth
from test_gpu_parity import colwise, dev, host, rel, tl  # noqa: F401

pytestmark = pytest.mark.gpu


def check_apply(tl, m, n, k, mb, tree):  # noqa: F811
    print(f"case m={m} n={n} k={k} mb={mb} tree={tree}", flush=True)
    A, B = synth.gaussian(m, n, seed=50 * n + k), synth.gaussian(m, k, seed=n + 7 * k)
    # the leading n rows of Q^T B (R's signs) and the others' norms do not
    # depend on the tree; the oracle's own trees are the uniform ones
    orc = oracle.TSQR(A, mb=mb, tree=tree if tree in (0, 2, 4, 8) else 2)
    f = tl.factor(dev(A), row_block=mb, tree=tree)
    Bd = dev(B)
    f.apply_qt_(Bd)
    C, Co = host(Bd), orc.apply_qt(B)
    assert rel(C[:n], Co[:n]) <= 1e-12
    colwise(C[:n], Co[:n], 1e-12, scale=np.linalg.norm(B, axis=0))
    assert np.allclose(np.linalg.norm(C[n:], axis=0), np.linalg.norm(Co[n:], axis=0), rtol=1e-11,
                       atol=1e-13 * np.linalg.norm(B))
    f.apply_q_(Bd)
    assert rel(host(Bd), B) <= 1e-13


# 2305 rows in blocks of 256: 9 domains, the last merged or short; odd, so no
# 16-byte column starts
@pytest.mark.parametrize("k", [1, 2, 15, 16, 17, 33, 64, 65])
@pytest.mark.parametrize("n", [1, 8, 15, 16, 17, 32, 33, 48, 49, 63, 64])
def test_block_edges(tl, n, k):  # noqa: F811
    check_apply(tl, 2305, n, k, 256, 2)


@pytest.mark.parametrize("k", [1, 20, 40])
@pytest.mark.parametrize("n", [5, 40, 64, 100])
@pytest.mark.parametrize("tree", [0, 2, 4, 8, "xcd"])
def test_tree_shapes(tl, tree, n, k):  # noqa: F811
    # 12 domains of several chunks, an even height: 16-byte column starts
    check_apply(tl, 6400, n, k, 520, tl.TREE_XCD if tree == "xcd" else tree)
