"""Few columns through a mixed-precision factor of several panels: the error of
Q Q^T B does not depend on whether the domains are fewer or more than the
compute units (256).  What is compared is ||B - Q Q^T B|| / ||B||, the sum of
some 1e6 FP32 roundings, for two heights 1 % apart with the same domains and
columns of the same distribution: the two agree to a few percent (its relative
spread is about one over the root of the number of rows, and the height itself
enters by its square root at most), so 1.25 is allowed; W, Z and the running
top rows in FP32 on one side make it about 2.

More than 16 columns go through the chained form, whose chain over T is FP32;
in domains of 64 rows its error per column was 1.8 times (16 columns of V) and
2.35 times (40) that of few columns while the 64 products of W met in sums of 16,
2.8 and 3.0 times with all of them in one chain: the line is drawn between."""
import pytest
import torch

from test_gpu_mixed import tl  # noqa: F401

pytestmark = pytest.mark.gpu


def error(tl, P, mb, n, k):  # noqa: F811
    m = P * mb
    g = torch.Generator(device="cuda").manual_seed(n + k)
    A = torch.randn((n, m), generator=g, device="cuda", dtype=torch.float64).t()
    B0 = torch.randn((k, m), generator=g, device="cuda", dtype=torch.float64).t()
    f = tl.factor(A, prec=tl.MIXED, row_block=mb)
    B = B0.t().clone().t()
    f.apply_qt_(B)
    f.apply_q_(B)
    e = float((B - B0).norm() / B0.norm())
    print(f"case mixed {m} x {n}, {P} domains, {k} columns: error {e:.2e}", flush=True)
    return e


@pytest.mark.parametrize("n,mb,k", [(128, 256, 1), (128, 1024, 2), (72, 256, 16)])
def test_same_error_on_both_sides_of_the_compute_units(tl, n, mb, k):  # noqa: F811
    few, many = error(tl, 255, mb, n, k), error(tl, 258, mb, n, k)
    assert many <= 1.25 * few


@pytest.mark.parametrize("n,most", [(16, 2.25), (40, 2.65)])
def test_low_domains_sum_by_tiles(tl, n, most):  # noqa: F811
    few, more = error(tl, 3125, 64, n, 16), error(tl, 3125, 64, n, 17)
    assert more <= most * few
