"""The timing pass under link occupancy and with costs per micro-batch at the device counts where its lanes and segments
can go wrong, with costs of one and of two bytes, and batches in which segments take further candidates."""
import numpy as np
import pytest

import workloads
from gpu_common import check_batch
from test_gpu_lists import spec_of
from workloads.problem import chain_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("links", [False, True])
@pytest.mark.parametrize("largest", [None, 255, 256])
@pytest.mark.parametrize("D,v,m", [(1, 2, 5), (2, 1, 33), (5, 4, 9), (17, 2, 8), (22, 1, 7), (33, 2, 4), (64, 1, 3)])
def test_device_counts(D, v, m, largest, links):
    if largest is None and not links:
        return   # the plain form
    prob = chain_problem(D, m, v=v, f=30, b=50, w=20, comm=45, mem_cap=max(2, D // 2))
    words = workloads.generate(spec_of(prob, 150, D), threads=8)
    words = np.tile(words, (1 + 20000 // (150 * D), 1, 1))
    table = None
    if largest is not None:
        table = np.random.default_rng(D).integers(0, largest + 1, (8, prob.n_stages, m)).astype(np.int32)
        table[1:, 0, 0] = largest
        table[7] = table[1]   # (kinds that share a block of the table)
    check_batch(prob, words, 8, f"D={D}", kernels=("slots",), links=links, dur_mb=table)
