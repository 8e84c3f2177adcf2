"""The timing pass hands out candidates: as many as there are segments, one more or fewer, several rounds of them, candidates
short enough to be drawn several at a time and long ones drawn one by one."""
import numpy as np
import pytest
import torch

import oracle
import paper_2510_05112_amd as fp
import workloads
from workloads.problem import chain_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,v,m,factors", [(16, 1, 6, (1, 2, 3.3)), (2, 2, 3, (1, 1.7)), (31, 4, 48, (1, 1.4))])
def test_batches_around_the_number_of_segments(D, v, m, factors):
    prob = chain_problem(D, m, v=v, f=3, b=5, w=2, comm=1, mem_cap=D)
    spec = workloads.Spec(0, prob, 64, -(-3 * v * m // 8) * 8, 8, cap_units=D, seed=D, deadlock_per_mille=60)
    base = workloads.generate(spec, threads=8)
    ref = oracle.evaluate(prob, base, threads=8)
    h = fp.Problem(prob, spec.stride, device=0)
    cpw = h.info()["candidates_per_wave"]
    segments = torch.cuda.get_device_properties(0).multi_processor_count * 16 * cpw   # (at most: sixteen wavefronts per compute unit)
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
