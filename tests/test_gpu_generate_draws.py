"""How the generator's segments come by their sets: class by class or in plain order, on both sides of the line between
them, in batches that do not divide evenly; and that short sets do not wait for the draws."""
import numpy as np
import pytest

from test_genoracle import random_policies, stride_for
from test_gpu_generate import check
from test_gpu_generate_evaluate import placed_chain
from test_gpu_generate_slide import check_slide

pytestmark = pytest.mark.gpu


# one wavefront per compute unit: 256 x (64 / p) segments; p, v, m: 15 x 3 v m (1 + v) steps, by class from one per segment on
# (lists; the sliding form has fewer sets in a wavefront here, and its orders in test_gpu_generate_slide_shared.py)
@pytest.mark.parametrize("p,v,m,sets_per_segment", [(20, 2, 2, 2.5), (20, 2, 3, 1.9), (20, 2, 3, 2.0), (20, 2, 3, 2.7), (20, 1, 8, 2.1),
                                                    (20, 1, 9, 2.1), (40, 4, 4, 1.3), (40, 4, 4, 6.1), (7, 3, 5, 3.3), (7, 3, 4, 3.3)])
def test_both_orders(p, v, m, sets_per_segment, monkeypatch):
    monkeypatch.setenv("FPSCHED_GEN_WAVES", "1")
    prob = placed_chain(p, v, m, 1, seed=p)
    n = int(256 * (64 // p) * sets_per_segment)
    rng = np.random.default_rng(n)
    pol, inf = random_policies(rng, n, prob, rng.random(n) < 0.5)
    check(prob, pol, inf, stride_for(prob), f"p{p}")
    check_slide(prob, pol, inf, f"p{p}")


def test_short_sets_do_not_wait_for_the_draws():
    """65,536 sets, 24,576 at a time: 7 times as long as 24,576; 23 times when each was drawn class by class."""
    import torch
    import paper_2510_05112_amd as fp
    import workloads
    prob = placed_chain(8, 1, 8, 1, seed=8)
    stride = stride_for(prob)
    h = fp.Problem(prob, stride, device=0)

    def best_time(n):
        pol, inf = (torch.from_numpy(x).cuda() for x in workloads.policy_sets(prob, n, 1))
        out, ws = h.generate(pol, inf, stride), h.alloc_workspace(n, 0)
        times = []
        for _ in range(8):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            h.generate(pol, inf, stride, out=out, workspace=ws)
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b))
        return min(times)

    assert best_time(65536) < 12 * best_time(24576)
    h.close()
