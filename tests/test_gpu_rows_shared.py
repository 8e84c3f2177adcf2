"""The order pass where four lanes read each other's rows (more than eight wavefronts of rows per compute unit, rows of 64
words and more): rows that end in every part of a request, batches whose last rows leave lanes of the four without one,
one to four stages per device, with and without W items, blocks that are drawn.  (That these batches are launched as that form:
test_host_launches.py.)"""
import numpy as np
import pytest
import torch

import oracle
import paper_2510_05112_amd as fp
import workloads
from gpu_common import assert_same, check_batch
from workloads.problem import chain_problem

pytestmark = pytest.mark.gpu


PADDINGS = (0, 8, 16, 24)
EVALUATED = ((1, 1, 22, 140001), (3, 1, 27, 140002), (5, 2, 11, 140005), (7, 4, 6, 140007), (2, 1, 40, 140002))   # devices, stages per device, micro-batches, rows
WITHOUT_W = ((3, 1, 27, 140002), (5, 2, 11, 140005), (7, 4, 6, 140007))
DRAWN = (9, 2, 12, 64 * 3072 * 10)


def problem_of(D, v, m, padding):
    """... and its rows' words"""
    return chain_problem(D, m, v=v, f=3, b=5, w=2, comm=1, mem_cap=max(2, D)), -(-3 * v * m // 8) * 8 + padding


def batch(D, v, m, padding, n_rows, seed):
    prob, stride = problem_of(D, v, m, padding)
    spec = workloads.Spec(0, prob, 200, stride, 8, cap_units=max(2, D), seed=seed, deadlock_per_mille=60)
    base = workloads.generate(spec, threads=8)
    return prob, np.tile(base, (-(-n_rows // (200 * D)), 1, 1))[:-(-n_rows // D)]


@pytest.mark.parametrize("padding", PADDINGS)
@pytest.mark.parametrize("D,v,m,n_rows", EVALUATED)
def test_rows_of_four_lanes(D, v, m, n_rows, padding):
    prob, words = batch(D, v, m, padding, n_rows, D + padding)
    assert words.shape[2] >= 64
    check_batch(prob, words, 8, f"{D} {v} {m} + {padding}", threads=16, kernels=("slots",))


@pytest.mark.parametrize("D,v,m,n_rows", WITHOUT_W)
def test_without_w_items(D, v, m, n_rows):
    prob, words = batch(D, v, m, 8, n_rows, D)
    stride = words.shape[2]
    h = fp.Problem(prob, stride, device=0)
    got = h.wslide(torch.from_numpy(words.view(np.int16)).cuda(), stride)
    torch.cuda.synchronize()
    ref = oracle.wslide(prob, words[:200], stride, threads=16)
    for at in range(0, len(words), 200):   # (copies of the first 200)
        part = {name: got[name][at:at + 200].cpu().numpy() for name in ("makespan", "idle", "peak", "flags")}
        assert_same(part, {name: ref[name][:len(part["flags"])] for name in part}, f"{D} {v} {m} from {at}")
    h.close()


def test_blocks_that_are_drawn():
    prob, words = batch(*DRAWN[:3], 8, DRAWN[3], 3)
    check_batch(prob, words[:-1], 16, "more than eight blocks to a wavefront", threads=16, kernels=("slots",))
