"""Order pass, where its rows stand in LDS: in columns (a power of two of them, with the devices over and over where they are one
too and a wavefront walks more than one block of rows), and device by device where columns would cost a wavefront."""
import numpy as np
import pytest

import workloads
from gpu_common import check_batch
from workloads.problem import chain_problem

pytestmark = pytest.mark.gpu


def batch(D, v, m, n):
    prob = chain_problem(D, m, v=v, f=3, b=5, w=2, comm=2, mem_cap=max(2, D // 2))
    prob.dur[:] = prob.dur * np.random.default_rng(D * 8 + v).integers(1, 6, prob.dur.shape)
    stride = -(-3 * v * m // 8) * 8 + 8
    spec = workloads.Spec(0, prob, n, stride, 8, cap_units=max(2, D // 2), seed=D + v, deadlock_per_mille=50)
    return prob, workloads.generate(spec, threads=8)


@pytest.mark.parametrize("D,v", [(1, 1), (2, 4), (4, 2), (5, 3), (17, 1), (32, 2), (33, 2), (48, 1), (63, 1), (64, 1)])
@pytest.mark.parametrize("blocks", [1, 2])
def test_columns(D, v, blocks):
    n = 150 if blocks == 1 else -(-200_000 // D)   # (more rows than 64 for each of twelve wavefronts on 256 compute units)
    prob, words = batch(D, v, 3, n)
    check_batch(prob, words, 8, f"D={D} v={v} n={n}", kernels=("slots",))


@pytest.mark.parametrize("D,v,m", [(3, 1, 236), (5, 2, 98), (11, 4, 47), (23, 2, 86), (33, 1, 140), (40, 2, 70)])
def test_device_by_device(D, v, m):
    prob, words = batch(D, v, m, 40)
    check_batch(prob, words, 8, f"D={D} v={v} m={m}", kernels=("slots",))
