"""The timing pass's requests: lists that end at every piece of a request of 64 (or 32) bytes, in rows that they fill or
that go on for up to three further pieces, in the plain form and in one that requests less at a time."""
import numpy as np
import pytest

import workloads
from gpu_common import check_batch
from workloads.problem import chain_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("words", [8, 16, 24, 32, 40, 48, 56, 64, 72, 104])
@pytest.mark.parametrize("padding", [0, 8, 16, 24])
def test_lists_end_at_every_piece(words, padding):
    prob = chain_problem(3, words // 2, v=1, f=2, b=4, w=None, comm=1)
    spec = workloads.Spec(0, prob, 400, words + padding, 8, cap_units=2, seed=words, deadlock_per_mille=30)
    batch = np.tile(workloads.generate(spec, threads=4), (3, 1, 1))
    check_batch(prob, batch, 8, f"{words} + {padding}", kernels=("slots",))
    check_batch(prob, batch, 8, f"{words} + {padding}, links", kernels=("slots",), links=True)
