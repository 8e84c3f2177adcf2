"""The timing pass hands out candidates: as many as there are segments, one more or fewer, several rounds of them, candidates
short enough to be drawn a segment's worth at a time, by share, and long ones drawn one by one.  (That the wavefronts and draws are
those said here: test_host_launches.py.)"""
import numpy as np
import pytest
import torch

import oracle
import paper_2510_05112_amd as fp
import workloads
from workloads.problem import chain_problem

pytestmark = pytest.mark.gpu


# devices, stages per device, micro-batches, wavefronts per compute unit, candidates of a draw at least and at most, batches per segment
CASES = ((16, 1, 6, 28, 8, 8, (1, 2, 3.3)), (2, 2, 3, 22, 64, 64, (1, 1.7)), (16, 2, 32, 20, 4, 8, (1, 2.3, 4)), (31, 4, 48, 20, 1, 1, (1, 1.4)))


def problem_of(D, v, m):
    """... and its rows' words"""
    return chain_problem(D, m, v=v, f=3, b=5, w=2, comm=1, mem_cap=D), -(-3 * v * m // 8) * 8


@pytest.mark.parametrize("D,v,m,waves,least,most,factors", CASES)
def test_batches_around_the_number_of_segments(D, v, m, waves, least, most, factors):
    prob, stride = problem_of(D, v, m)
    spec = workloads.Spec(0, prob, 64, stride, 8, cap_units=D, seed=D, deadlock_per_mille=60)
    base = workloads.generate(spec, threads=8)
    ref = oracle.evaluate(prob, base, threads=8)
    h = fp.Problem(prob, spec.stride, device=0)
    segments = torch.cuda.get_device_properties(0).multi_processor_count * waves * h.info()["candidates_per_wave"]
    ops = torch.from_numpy(base.view(np.int16)).cuda()
    for factor in factors:
        for more in (-1, 0, 1):
            n = int(segments * factor) + more
            res = h.evaluate(ops[torch.arange(n, device="cuda") % 64])
            torch.cuda.synchronize()
            for name in ("flags", "makespan", "idle", "peak"):
                want = torch.from_numpy(ref[name]).cuda()[torch.arange(n, device="cuda") % 64]
                assert torch.equal(res[name], want), (name, n)
    h.close()
