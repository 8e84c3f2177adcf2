"""The timing pass where stages have second inputs and outputs: outputs that continue one, both or none of the inputs'
classes, in lists that are kept, dropped and recomputed, with more candidates than a launch has segments."""
import numpy as np
import pytest

from gpu_common import check_batch
from helpers import batch_from_lists, dag_problem, perturb, random_valid_lists

pytestmark = pytest.mark.gpu

# edges, stages, device of each stage
SHAPES = {
    "two in, two out": ([(0, 2), (1, 2), (2, 3), (2, 4)], 5, [0, 1, 2, 3, 4]),
    "one in, two out": ([(0, 1), (1, 2), (1, 3)], 4, [0, 1, 2, 3]),
    "two in, none out": ([(0, 2), (1, 2)], 3, [0, 1, 2]),
    "diamonds, two stages to a device": ([(0, 1), (0, 2), (1, 3), (2, 3), (3, 4), (3, 5), (4, 6), (5, 6)], 7, [0, 1, 2, 3, 0, 1, 2]),
    "skips": ([(0, 1), (1, 2), (2, 3), (0, 2), (1, 3)], 4, [0, 1, 2, 0]),
}


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("m", [1, 7, 33])
def test_second_edges(shape, m):
    edges, n_stages, placement = SHAPES[shape]
    rng = np.random.default_rng(m)
    prob = dag_problem(edges, n_stages, placement, max(placement) + 1, m=m, has_w=1, seed=m)
    lists = []
    for t in range(24):
        base = random_valid_lists(prob, rng, 0.3 * (t % 2), 0.3 * ((t // 2) % 2))
        lists += [base, perturb(base, rng, 1 + t % 3)]
    words = batch_from_lists(lists)
    check_batch(prob, words, 7, shape, kernels=("slots",))
    check_batch(prob, words, 7, shape + ", links", kernels=("slots",), links=True)
    if m == 7:
        check_batch(prob, np.tile(words, (2000, 1, 1)), 7, shape + ", many", kernels=("slots",))
