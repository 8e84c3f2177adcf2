"""The copy engine's two passes at depths beyond those with few registers (four transfers kept, or seven): results against the oracle
in both forms, on either side of the lines between them (which form each batch is launched as: test_host_launches.py), lists whose
transfers fill the engine."""
import numpy as np
import pytest

import oracle
from gpu_common import assert_same
from helpers import batch_from_lists, perturb, random_valid_lists
from test_gpu_copy import FORM_LISTS, gpu_copy, resident_of, transfer_problems
from workloads.problem import L, O, chain_problem

pytestmark = pytest.mark.gpu


DEPTHS = (4, 5, 7)


def form_problems():
    long_rows = [chain_problem(5, 20, v=2, f=2, b=3, w=1, comm=1), chain_problem(3, 36, v=1, f=2, b=3, w=1, comm=1), chain_problem(4, 6, v=4, f=3, b=4, w=2, comm=1)]
    for prob in long_rows:
        prob.dur[O], prob.dur[L] = 3, 2
    return transfer_problems() + long_rows


@pytest.mark.parametrize("depth", DEPTHS)
@pytest.mark.parametrize("slow", [1, 60])
def test_deep_engines(depth, slow, monkeypatch, capfd):
    monkeypatch.setenv("FPSCHED_VERBOSE", "1")
    rng = np.random.default_rng(100 * depth + slow)
    for i, prob in enumerate(form_problems()):
        prob.dur[O] = prob.dur[O] * slow   # (transfers that take longer than what runs beside them: the engine is full)
        prob.dur[L] = prob.dur[L] * slow
        lists = []
        for t in range(FORM_LISTS // 2):
            base = random_valid_lists(prob, rng, 0.3 * (t % 2), 0.4 + 0.3 * ((t // 2) % 2))
            lists += [base, perturb(base, rng, 1 + t % 3)]
        words = batch_from_lists(lists)
        ref = oracle.evaluate_copy(prob, words, depth=depth, threads=8)
        copies = resident_of(prob, words.shape[2], depth, capfd) // len(words) + 1
        for times in (1, copies):
            out, _ = gpu_copy(prob, np.tile(words, (times, 1, 1)), depth)
            assert_same(out, {name: np.tile(a, (times,) + (1,) * (a.ndim - 1)) for name, a in ref.items()}, f"problem {i}, {times} times, depth {depth}")
