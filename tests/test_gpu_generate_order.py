"""The generator where a batch has more sets than the launch has segments (here in plain order; by class:
test_gpu_generate_draws.py) on device counts that leave lanes of a wavefront over, and the sliding form where stashes and
item rings wrap."""
import numpy as np
import pytest

from test_genoracle import NO_LIMIT, random_policies, stride_for
from test_gpu_generate import check
from test_gpu_generate_evaluate import placed_chain
from test_gpu_generate_slide import check_slide

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p,v,m,n", [(3, 1, 2, 65001), (20, 2, 3, 9999), (40, 4, 2, 3333), (31, 2, 16, 8000)])
def test_more_sets_than_segments(p, v, m, n):
    prob = placed_chain(p, v, m, 1, seed=p)
    rng = np.random.default_rng(n)
    pol, inf = random_policies(rng, n, prob, rng.random(n) < 0.5)
    check(prob, pol, inf, stride_for(prob), f"p{p}")
    check_slide(prob, pol, inf, f"p{p}")


@pytest.mark.parametrize("p,v,m", [(1, 1, 90), (2, 2, 80), (32, 2, 64), (3, 4, 33), (2, 3, 100), (20, 4, 16)])
def test_deep_stashes(p, v, m):
    prob = placed_chain(p, v, m, 1, seed=v)
    rng = np.random.default_rng(m)
    pol, inf = random_policies(rng, 60, prob, rng.random(60) < 0.5)
    inf[::2] = NO_LIMIT
    check_slide(prob, pol, inf, f"p{p} v{v} m{m}")
