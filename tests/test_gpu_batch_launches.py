"""tsqr_batch_launches is the number of launches a run enqueues: compared with
the launches that the library's own kernel timing sees in a plain run, before
and after the first run (a plan's count does not change by running it)."""
import pytest
import torch

from test_gpu_batch import tl  # noqa: F401

pytestmark = pytest.mark.gpu


# (m, n) of the matrices; which are mixed
@pytest.mark.parametrize("shapes,precs", [
    ([(300, 8)], [0]),                                            # one domain, no tree
    ([(20000, 8), (9000, 16)], [0, 0]),                           # narrow, several domains
    ([(20000, 8), (9000, 32), (30000, 64)], [0, 1, 0]),           # every slot width, one mixed
    ([(500, 64), (700, 20)], [1, 1]),                             # mixed, one domain each
])
def test_count_is_what_a_run_enqueues(tl, shapes, precs):  # noqa: F811
    print(f"case launches {shapes} {precs}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(3)
    As = [torch.randn((n, m), generator=g, device="cuda", dtype=torch.float64).t() for m, n in shapes]
    bs = [torch.randn(m, generator=g, device="cuda", dtype=torch.float64) for m, _ in shapes]
    B = tl.Batch(As, bs, precs)
    before = B.launches()
    tl.prof_enable(True)
    try:
        B.run(use_graph=False)
        torch.cuda.synchronize()
        seen = sum(c for c, _ in tl.prof_query().values())
    finally:
        tl.prof_enable(False)
    assert before == seen
    assert B.launches() == seen
