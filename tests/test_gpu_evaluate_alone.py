"""Both passes of the list evaluation in one launch: batches of the sizes at which the one launch begins, a wavefront gets another
candidate, a SIMD its second wavefront, and the two launches take over, with lists that deadlock, stop and fill their rows, against
the oracle.  The batches are copies of a few candidates, so that the oracle has these only to do."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from gpu_common import assert_same, gpu_evaluate
from helpers import two_tower_problem
from test_gpu_row_columns import batch

pytestmark = pytest.mark.gpu


def sizes(D, short):
    cu = torch.cuda.get_device_properties(0).multi_processor_count
    most = min(64 // D, 64 // ((D + 1) // 2)) * cu
    n = {1, 63, 64, 4 * cu, 4 * cu + 1, 4 * most - 1, 4 * most, 4 * most + 1, 8 * most, 8 * most + 1}
    return sorted(x for x in n if x * D <= (1 << 18 if short else 1 << 17))


def check(prob, words, what, short=True):
    ref = oracle.evaluate(prob, words, threads=8)
    for n in sizes(prob.n_devices, short):
        which = np.arange(n) % len(words)
        gpu, _ = gpu_evaluate(prob, words[which], kernel="slots")
        assert_same(gpu, {name: v[which] for name, v in ref.items()}, f"{what} n={n}")


@pytest.mark.parametrize("D,v,m", [(1, 1, 3), (2, 2, 5), (3, 4, 4), (4, 1, 8), (7, 3, 5), (8, 2, 9), (12, 2, 7), (16, 2, 8), (24, 1, 9),
                                   (31, 2, 5), (32, 2, 6), (33, 1, 7), (64, 1, 5)])
def test_sizes_at_which_the_route_changes(D, v, m):
    prob, words = batch(D, v, m, n=70)
    check(prob, words, f"D={D} v={v}")
    prob, words = batch(D, v, m, (1 << 30) // (D * words.shape[2] * 26), n=70)
    check(prob, words, f"times of two words D={D} v={v}")


@pytest.mark.parametrize("D,v,m", [(8, 2, 32), (12, 2, 40), (32, 2, 30)])
def test_long_rows(D, v, m):
    prob, words = batch(D, v, m, n=70)
    check(prob, words, f"D={D} v={v} m={m}", short=False)


def test_second_edges():
    prob = two_tower_problem()
    spec = workloads.Spec(0, prob, 70, -(-3 * prob.n_microbatches * 4 // 8) * 8 + 8, 8, cap_units=6, seed=5, deadlock_per_mille=50)
    check(prob, workloads.generate(spec, threads=8), "two towers")


@pytest.mark.parametrize("D,m", [(2, 6), (6, 5)])
def test_sizes_at_which_a_compute_unit_has_one_wavefront(D, m):
    # (four stages per device: a wavefront has all of a compute unit's candidates, up to sixteen)
    cu = torch.cuda.get_device_properties(0).multi_processor_count
    prob, words = batch(D, 4, m, n=70)
    ref = oracle.evaluate(prob, words, threads=8)
    links = oracle.evaluate(prob, words, threads=8, links=True)
    for n in (cu, cu + 1, 3 * cu + 1, 4 * cu, 4 * cu + 1, 16 * cu - 1, 16 * cu, 16 * cu + 1):
        which = np.arange(n) % len(words)
        gpu, _ = gpu_evaluate(prob, words[which], kernel="slots")
        assert_same(gpu, {name: v[which] for name, v in ref.items()}, f"D={D} n={n}")
        gpu, _ = gpu_evaluate(prob, words[which], kernel="slots", links=True)
        assert_same(gpu, {name: v[which] for name, v in links.items()}, f"links D={D} n={n}")
