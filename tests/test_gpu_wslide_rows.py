"""The second kernel of the sliding pass in its two forms, a wavefront per row for few rows and a lane per row for many (beyond
12,288 rows, 16,384 on few devices, 24,576 where they are longer), on the same lists: long and short rows, chunks out of order,
waits of 2^16 time units and more, lists that stop early, rows of the new lists that are too short."""
import numpy as np
import pytest
import torch

import oracle
import paper_2510_05112_amd as fp
from helpers import batch_from_lists, perturb, random_valid_lists
from test_gpu_fuzz import random_problem
from workloads.problem import chain_problem

pytestmark = pytest.mark.gpu


def lists_of(prob, rng, n):
    lists = []
    for t in range(n):
        base = random_valid_lists(prob, rng, 0.3 * (t % 2), 0.3 * ((t // 2) % 2))
        lists += [base, perturb(base, rng, 1 + t % 3)]
        cut = [list(x) for x in base]
        d = int(rng.integers(prob.n_devices))
        cut[d] = cut[d][: len(cut[d]) // 2]
        lists.append(cut)
    return batch_from_lists(lists)


def check(prob, words, what):
    n, D, stride = words.shape
    many = -(-24600 // (n * D))
    h = fp.Problem(prob, stride + 8, device=0)
    for stride_out in (stride + 8, max(8, stride // 2 // 8 * 8)):
        ref = oracle.wslide(prob, words, stride_out, threads=8)
        for copies in (1, many):
            ops = torch.from_numpy(np.tile(words, (copies, 1, 1)).view(np.int16)).cuda()
            out = h.wslide(ops, stride_out)
            torch.cuda.synchronize()
            for name in ("ops", "makespan", "idle", "peak", "flags"):
                got = out[name].cpu().numpy()
                got = got.view(np.uint16) if name == "ops" else got
                assert np.array_equal(got, np.tile(ref[name], (copies,) + (1,) * (ref[name].ndim - 1))), (what, stride_out, copies, name)
    h.close()


# (times stay below 2^24)
@pytest.mark.parametrize("devices,m,chunks,scale", [(1, 3, 1, 1), (2, 70, 1, 1), (3, 33, 2, 1), (5, 20, 3, 1), (4, 40, 4, 1), (33, 4, 1, 1),
                                                    (1, 3, 1, 4000), (2, 30, 1, 3000), (3, 12, 2, 1500), (2, 5, 4, 3000)])
def test_chains(devices, m, chunks, scale):
    rng = np.random.default_rng(devices * m)
    prob = chain_problem(devices, m, v=chunks, f=3 * scale, b=5 * scale, w=2 * scale, comm=min(scale, 30000))
    check(prob, lists_of(prob, rng, 6), f"{devices} x {m} x {chunks}, scale {scale}")


@pytest.mark.parametrize("seed", range(6))
def test_random_problems(seed):
    rng = np.random.default_rng(9000 + seed)
    done = 0
    while done < 5:
        prob = random_problem(rng)
        if prob.has_w:
            check(prob, lists_of(prob, rng, 6), f"seed {seed} problem {done}")
            done += 1
