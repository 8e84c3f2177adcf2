"""The generator's three forms at the ends of the policies' ranges: turns of one item and of more than there are, intervals of
one item, of the largest count a traversal state holds and beyond, one to four stages per actor, with and without W items."""
import numpy as np
import pytest

import test_gpu_generate
import test_gpu_generate_evaluate
import test_gpu_generate_slide
from test_genoracle import random_policies, stride_for
from workloads.problem import chain_problem

pytestmark = pytest.mark.gpu
MOST = 2**31 - 1


@pytest.mark.parametrize("chunks", [1, 2, 3, 4])
@pytest.mark.parametrize("w", [None, 2])
def test_extreme_policies(chunks, w):
    prob = chain_problem(5, 9, v=chunks, f=3, b=5, w=w, comm=2)
    rng = np.random.default_rng(chunks)
    n = 400
    pol, inf = random_policies(rng, n, prob, rng.random(n) < 0.5)
    units, intervals = [1, 2, MOST - 1, MOST], [0, 1, 2, 0x3ffe, 0x3fff, 0x4000, MOST]
    inter = pol[:, :, 0] == 2
    for column in (1, 2):
        pol[:, :, column] = np.where(inter, rng.choice(units, inter.shape), 1)
    for column in (4, 6):
        pol[:, :, column] = rng.choice(intervals, inter.shape)
    what = f"{chunks} stages per actor, w {w}"
    test_gpu_generate.check(prob, pol, inf, stride_for(prob), what)
    test_gpu_generate_evaluate.check(prob, pol, inf, what)
    if w:
        test_gpu_generate_slide.check_slide(prob, pol, inf, what)
