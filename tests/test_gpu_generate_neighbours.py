"""Generator, two stages per actor: what an actor's stages wait for on one other actor, with the counters of both in one word
(halves in order and swapped, an actor with one stage, actors that wait for nothing, an actor that is its own neighbour, as many actors
as stages), on two other actors, and with more actors than stages; lists, results and results after sliding against the oracles."""
import numpy as np
import pytest

from helpers import dag_problem
from test_genoracle import random_policies
from test_gpu_generate import check, stride_for
from test_gpu_generate_evaluate import check as check_timed, placed_chain
from test_gpu_generate_slide import check_slide
from workloads.problem import chain_problem

pytestmark = pytest.mark.gpu


def problems():
    for D in (1, 2, 3, 8, 21, 32, 64):
        yield f"round the {D} devices", chain_problem(D, 5, v=2, f=3, b=4, w=2, comm=1)
    yield "up and down", placed_chain(5, 2, 6, 1, seed=1, circular=False)
    yield "one device with one stage", dag_problem([(s, s + 1) for s in range(6)], 7, [s % 4 for s in range(7)], 4, m=6)
    yield "two chains", dag_problem([(0, 1), (1, 2), (3, 4), (4, 5)], 6, [0, 1, 2, 0, 1, 2], 3, m=6)
    yield "two chains, halves swapped", dag_problem([(0, 4), (4, 2), (3, 1), (1, 5)], 6, [0, 1, 2, 0, 1, 2], 3, m=6)
    yield "as many devices as stages", dag_problem([(0, 2), (1, 3)], 4, [3, 3, 1, 1], 4, m=6)
    yield "three stages on four devices", dag_problem([(0, 2)], 3, [0, 0, 3], 4, m=6)
    yield "two stages on the last of 21 devices", dag_problem([(0, 1)], 2, [20, 20], 21, m=6)
    yield "forward from one actor, backward from two", dag_problem([(0, 2), (1, 3)], 4, [0, 0, 1, 2], 3, m=6)


@pytest.mark.parametrize("name,prob", [pytest.param(*p, id=p[0].replace(" ", "_")) for p in problems()])
def test_neighbours(name, prob):
    rng = np.random.default_rng(prob.n_devices)
    pol, inf = random_policies(rng, 140, prob, rng.random(140) < 0.5)
    check(prob, pol, inf, stride_for(prob), name)
    check_timed(prob, pol, inf, name)
    check_slide(prob, pol, inf, name)
