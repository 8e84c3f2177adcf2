"""First pass of the sliding pass on the two-pass evaluation (chains): rows that fill their stride or end at any piece of
it, weight-gradient words anywhere, twice, or out of range, lists that stop at an illegal op."""
import numpy as np
import pytest
import torch

import oracle
import paper_2510_05112_amd as fp
import workloads
from workloads.problem import W, chain_problem, pack_word

pytestmark = pytest.mark.gpu


def check(prob, words, stride_out):
    h = fp.Problem(prob, max(words.shape[2], stride_out), device=0)
    out = h.wslide(torch.from_numpy(np.ascontiguousarray(words).view(np.int16)).cuda(), stride_out)
    torch.cuda.synchronize()
    ref = oracle.wslide(prob, words, stride_out, threads=8)
    for name, want in ref.items():
        got = out[name].cpu().numpy()
        assert np.array_equal(got.view(np.uint16) if name == "ops" else got, want), name
    h.close()
    return ref


@pytest.mark.parametrize("m,v,padding", [(2, 1, 0), (8, 1, 0), (8, 1, 8), (16, 1, 0), (16, 1, 8), (24, 1, 24), (8, 2, 0), (8, 3, 16), (16, 4, 0),
                                         (5, 1, 1), (11, 2, 6)])
def test_rows_of_every_length(m, v, padding):
    prob = chain_problem(3, m, v=v, f=3, b=5, w=2, comm=2, mem_cap=2)
    spec = workloads.Spec(0, prob, 500, -(-(3 * m * v) // 8) * 8 + 8 * (padding // 8), 8, cap_units=2, seed=m, deadlock_per_mille=40)
    words = np.tile(workloads.generate(spec, threads=4), (4, 1, 1))
    ref = check(prob, words, spec.stride)
    assert ((ref["flags"] & 3) == 0).sum() > 1000


@pytest.mark.parametrize("seed", range(6))
def test_weight_gradient_words_anywhere(seed):
    rng = np.random.default_rng(seed)
    D, m, v = int(rng.integers(1, 8)), int(rng.integers(3, 20)), int(rng.integers(1, 3))
    prob = chain_problem(D, m, v=v, f=3, b=5, w=2, comm=3, mem_cap=4)
    spec = workloads.Spec(0, prob, 300, -(-(4 * m * v) // 8) * 8, 8, cap_units=3, seed=seed, deadlock_per_mille=0)
    words = workloads.generate(spec, threads=4)
    for c in range(len(words)):
        d = int(rng.integers(D))
        at = np.flatnonzero(words[c, d] >> 13 == W)
        what = int(rng.integers(4))
        if what == 1 and len(at):      # another item of the same kind
            words[c, d, rng.choice(at)] = pack_word(W, int(rng.integers(v)), int(rng.integers(m)))
        elif what == 2 and len(at):    # out of range: the list stops there
            words[c, d, rng.choice(at)] = pack_word(W, int(rng.integers(4)), int(rng.integers(m, 2048)))
        elif what == 3:                # in front of everything, more than there are
            row = words[c, d]
            n = min(int((row == 0).sum()), int(rng.integers(1, 9)))
            words[c, d] = np.concatenate([np.full(n, pack_word(W, 0, 0), np.uint16), row[:len(row) - n]])
    check(prob, words, spec.stride)
