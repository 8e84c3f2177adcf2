"""The sliding pass where the stash ring wraps, runs full and is left for the row: depths around its 128 entries, B items
in and out of order, both together."""
import numpy as np
import pytest

import oracle
import paper_2510_05112_amd as fp
from workloads.problem import B, F, W, chain_problem, pack_word

pytestmark = pytest.mark.gpu


def lists(m, v, order, wait):
    """Forward items, then B items in `order`; W items somewhere; gaps only where device 1 is waited for."""
    rows = []
    for d in range(2):
        words = [pack_word(F, c, j) for c in range(v) for j in range(m)]
        for i, j in enumerate(order):
            words += [pack_word(B, c, j) for c in reversed(range(v))]
            if i % wait == wait - 1:
                words += [pack_word(W, c, order[k]) for k in range(i - wait + 1, i + 1) for c in range(v)]
        words += [pack_word(W, c, order[k]) for k in range(len(order) // wait * wait, len(order)) for c in range(v)]
        rows.append(words)
    return rows


@pytest.mark.parametrize("m,v", [(127, 1), (129, 1), (64, 2), (65, 2), (200, 2), (40, 4), (300, 1)])
@pytest.mark.parametrize("shuffle", ["none", "late", "all"])
@pytest.mark.parametrize("w,comm", [(5, 7), (1, 7), (2, 29)])
def test_stash_depths(m, v, shuffle, w, comm):
    import torch
    rng = np.random.default_rng(m * v)
    prob = chain_problem(2, m, v=v, f=3, b=4, w=w, comm=comm, mem_cap=10**6)
    stride = -(-3 * m * v // 8) * 8
    order = np.arange(m)
    if shuffle == "late":
        order[m // 2:] = rng.permutation(order[m // 2:])
    elif shuffle == "all":
        order = rng.permutation(m)
    words = np.zeros((3, 2, stride), np.uint16)
    for k, wait in enumerate((1, 7, m)):
        for d, row in enumerate(lists(m, v, [int(j) for j in order], wait)):
            words[k, d, :len(row)] = row
    ref = oracle.wslide(prob, words, stride, threads=2)
    h = fp.Problem(prob, stride, device=0)
    got = h.wslide(torch.from_numpy(words.view(np.int16)).cuda(), stride)
    for name in ("flags", "makespan", "idle", "peak"):
        np.testing.assert_array_equal(got[name].cpu().numpy(), ref[name], err_msg=name)
    np.testing.assert_array_equal(got["ops"].cpu().numpy().view(np.uint16), ref["ops"])
    assert (ref["flags"] == 0).any()


@pytest.mark.parametrize("p,v,m,n", [(10, 4, 33, 400), (6, 4, 70, 200)])
def test_stashes_that_shrink_before_they_fill(p, v, m, n):
    import torch

    import workloads
    from test_genoracle import stride_for
    prob = chain_problem(p, m, v=v, f=10, b=11, w=9, comm=3, mem_cap=10**6)
    pol, inf = workloads.policy_sets(prob, n, p)
    st = stride_for(prob)
    words = oracle.generate(prob, pol, inf, st, threads=8)["words"]
    ref = oracle.wslide(prob, words, st, threads=8)
    got = fp.Problem(prob, st, device=0).wslide(torch.from_numpy(words.view(np.int16)).cuda(), st)
    np.testing.assert_array_equal(got["ops"].cpu().numpy().view(np.uint16), ref["ops"])
    np.testing.assert_array_equal(got["makespan"].cpu().numpy(), ref["makespan"])
