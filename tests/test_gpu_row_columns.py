"""Timing pass, where its rows stand in LDS: numbers of devices whose pairs divide the sixteen columns and others, one to four stages
per device (the odd devices' rows in the place of the third and fourth stage's, or behind), lists that end in a word with a chunk,
tables that leave no room for columns, and the forms with tables behind the rows.  (Batches of one candidate to a wavefront; of as
many as a large batch has: test_gpu_list_segments.py.)"""
import numpy as np
import pytest

import workloads
from gpu_common import check_batch
from workloads.problem import W, chain_problem

pytestmark = pytest.mark.gpu


def batch(D, v, m, scale=1, n=200):
    prob = chain_problem(D, m, v=v, f=3, b=5, w=2, comm=2, mem_cap=max(2, D // 2))
    rng = np.random.default_rng(D * 8 + v)
    prob.dur[:] = prob.dur * rng.integers(1, 6, prob.dur.shape) * scale
    stride = -(-3 * v * m // 8) * 8 + 8
    spec = workloads.Spec(0, prob, n, stride, 8, cap_units=max(2, D // 2), seed=D + v, deadlock_per_mille=50)
    words = workloads.generate(spec, threads=8)
    ends = (words >> 13) == 0
    words[ends] = rng.integers(0, 1 << 13, int(ends.sum()), dtype=np.uint16)   # (a list ends whatever the word's other bits are)
    assert int(words.max()) >> 13 == W
    return prob, words


@pytest.mark.parametrize("D", [1, 2, 3, 4, 5, 7, 8, 12, 15, 16, 31, 32])
@pytest.mark.parametrize("v", [1, 2, 3, 4])
def test_rows_of_every_device(D, v):
    prob, words = batch(D, v, 6)
    check_batch(prob, words, 8, f"D={D} v={v}", kernels=("slots",))
    costs = workloads.microbatch_costs(prob, D)
    check_batch(prob, words, 8, f"links D={D} v={v}", kernels=("slots",), links=True)
    check_batch(prob, words, 8, f"links, costs D={D} v={v}", kernels=("slots",), links=True, dur_mb=costs)
    prob, words = batch(D, v, 6, (1 << 30) // (D * words.shape[2] * 26))
    check_batch(prob, words, 8, f"times of two words D={D} v={v}", kernels=("slots",))


@pytest.mark.parametrize("D,v,m", [(16, 4, 96), (8, 3, 120)])
def test_without_room_for_columns(D, v, m):
    prob, words = batch(D, v, m, n=40)
    check_batch(prob, words, 8, f"D={D} v={v} m={m}", kernels=("slots",))
