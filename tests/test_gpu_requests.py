"""The timing pass's requests: lists that end at every piece of a request of 64 (or 32) bytes, in rows that they fill or
that go on for up to three further pieces, in the plain form and in one that requests less at a time."""
import numpy as np
import pytest

import oracle
import paper_2510_05112_amd as fp
import workloads
from gpu_common import assert_same, check_batch, gpu_evaluate
from workloads.problem import B, F, L, O, chain_problem, pack_word

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("words", [8, 16, 24, 32, 40, 48, 56, 64, 72, 104])
@pytest.mark.parametrize("padding", [0, 8, 16, 24])
def test_lists_end_at_every_piece(words, padding):
    prob = chain_problem(3, words // 2, v=1, f=2, b=4, w=None, comm=1)
    spec = workloads.Spec(0, prob, 400, words + padding, 8, cap_units=2, seed=words, deadlock_per_mille=30)
    batch = np.tile(workloads.generate(spec, threads=4), (3, 1, 1))
    check_batch(prob, batch, 8, f"{words} + {padding}", kernels=("slots",))
    check_batch(prob, batch, 8, f"{words} + {padding}, links", kernels=("slots",), links=True)


@pytest.mark.parametrize("beyond", [0, 8])
@pytest.mark.parametrize("scale", [1, 20])
def test_rows_as_long_as_positions_go(scale, beyond):
    """One device offloads and reloads its activation until its list fills the longest row that the timing pass takes (times of 24
    bits, and beyond), or the first one that the table kernel does; the same list without its last item is incomplete."""
    stride = (1 << 23) - 32 + beyond
    prob = chain_problem(1, 1, v=1, f=scale, b=scale)
    prob.dur[O], prob.dur[L] = scale, scale
    words = np.zeros((2, 1, stride), np.uint16)
    words[:, 0, 0] = pack_word(F, 0, 0)
    words[:, 0, 1:-1:2] = pack_word(O, 0, 0)
    words[:, 0, 2:-1:2] = pack_word(L, 0, 0)
    words[0, 0, -1] = pack_word(B, 0, 0)
    out, _ = gpu_evaluate(prob, words)
    assert_same(out, oracle.evaluate(prob, words), f"{scale} {stride}")
    assert out["makespan"][0] == scale * stride and out["flags"][1] == fp.FLAG_INCOMPLETE
