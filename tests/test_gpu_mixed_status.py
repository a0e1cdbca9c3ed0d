"""The status word of mixed-precision solves on well-conditioned problems.

Gaussian matrices are refined to rounding by one or two corrections, and a
first correction lands on either side of 1e-7 by FP32's rounding.  The status
word must not tell the two apart: 0 for every one, and the true backward error
eta = ||A^T (b - A x)|| / (||A||_F (||A||_F ||x|| + ||b - A x||)) at most 1e-12
(the bound that the status word stands for).  With a rule that lets the first
correction end a column, about one matrix in 25 of 5000 x 8 reports -3.
"""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tl():
    import paper_0912_2572_amd as t
    t.lib()
    assert torch.cuda.is_available(), "GPU test run without a GPU"
    return t


def gauss(g, m, n):
    return torch.randn((n, m), generator=g, device="cuda", dtype=torch.float64).t()


def eta(A, x, b):
    r, nA = b - A @ x, A.norm()
    return float((A.t() @ r).norm() / (nA * (nA * x.norm() + r.norm())))


@pytest.mark.parametrize("n,m,count", [(8, 5000, 256), (16, 20000, 128), (32, 5000, 128)])
def test_gaussian_batches_report_zero(tl, n, m, count):
    for seed in range(3):
        print(f"case mixed batch {count} of {m} x {n}, seed {seed}", flush=True)
        g = torch.Generator(device="cuda").manual_seed(1000 * n + seed)
        As = [gauss(g, m, n) for _ in range(count)]
        bs = [gauss(g, m, 1).reshape(-1) for _ in range(count)]
        B = tl.Batch(As, bs, [1] * count)
        B.run(use_graph=False)
        torch.cuda.synchronize()
        assert [int(B.info(i).item()) for i in range(count)] == [0] * count
        assert max(eta(A, B.x(i), b) for i, (A, b) in enumerate(zip(As, bs))) <= 1e-12


def test_gaussian_single_solves_report_zero(tl):
    m, n, k = 5000, 8, 4
    for seed in range(40):
        g = torch.Generator(device="cuda").manual_seed(seed)
        A, b = gauss(g, m, n), gauss(g, m, k)
        print(f"case mixed solve {m} x {n}, {k} right-hand sides, seed {seed}", flush=True)
        f = tl.factor(A, prec=tl.MIXED, lsq_max_rhs=k)
        for c in range(k):          # one at a time: a column's end does not wait for another's
            X, res, info = f.lsq(b[:, c:c + 1], A=A)
            assert int(info.item()) == 0
            assert float(f.backward_error(1).item()) <= 1e-12


def test_zero_right_hand_side_in_a_batch(tl):
    """x = 0 ends a column at once; its residual norm is still computed."""
    g = torch.Generator(device="cuda").manual_seed(5)
    As = [gauss(g, 3000, 16) for _ in range(2)]
    bs = [torch.zeros(3000, dtype=torch.float64, device="cuda"), gauss(g, 3000, 1).reshape(-1)]
    B = tl.Batch(As, bs, [1, 1])
    B.run(use_graph=False)
    torch.cuda.synchronize()
    assert [int(B.info(i).item()) for i in range(2)] == [0, 0]
    assert float(B.x(0).abs().max()) == 0.0 and float(B.resid(0).item()) == 0.0
