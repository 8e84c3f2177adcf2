"""The timing pass with as many candidates in a wavefront as a large batch has, in every form: batches beyond a candidate for each
SIMD (forms with two launches) and beyond those that one launch takes (plain model), copies of a few candidates, so that the oracle
has these only to do.  Rows in columns and as in the image, of one to four stages per device.  (That these batches are launched so:
test_host_launches.py.)  And the one launch where the order rows stand device by device."""
import numpy as np
import pytest
import torch

import oracle
import paper_2510_05112_amd as fp
import workloads
from gpu_common import assert_same, gpu_evaluate
from helpers import batch_from_lists, random_slot_sync_problem
from test_gpu_check_columns import batch as order_batch
from test_gpu_row_columns import batch
from test_gpu_sync_forms import lists_of

pytestmark = pytest.mark.gpu

SPREAD = 4 * 256        # candidates of 256 compute units up to which a wavefront of a form with two launches has a SIMD's share
ROWS = [(D, v, m) for D, m in ((1, 12), (2, 12), (3, 20), (4, 20), (5, 10), (7, 20), (8, 20), (12, 8), (15, 20), (16, 30), (31, 10), (32, 20)) for v in (1, 2, 3, 4)]
DEVICE_BY_DEVICE = ((5, 2, 98), (11, 4, 47), (23, 2, 86), (40, 2, 70))   # devices, stages per device, micro-batches


def beyond_one_launch(D, room):
    return 8 * min(64 // D, room) * 256 + 77


def copies_same(prob, words, n, ref, what, **model):
    which = np.arange(n) % len(words)
    gpu, _ = gpu_evaluate(prob, words[which], kernel="slots", **model)
    assert_same(gpu, {name: v[which] for name, v in ref.items()}, what)


def times_of_two_words(D, stride):
    return (1 << 30) // (D * stride * 26)


@pytest.mark.parametrize("D,v,m", ROWS)
def test_rows(D, v, m):
    prob, words = batch(D, v, m, n=70)
    ref = oracle.evaluate(prob, words, threads=8)
    h = fp.Problem(prob, words.shape[2], device=0)
    n = beyond_one_launch(D, h.info()["candidates_per_wave"])
    h.close()
    copies_same(prob, words, n, ref, f"D={D} v={v}")
    costs = workloads.microbatch_costs(prob, D)
    for model in (dict(links=True), dict(dur_mb=costs), dict(links=True, dur_mb=costs)):
        copies_same(prob, words, SPREAD + 300, oracle.evaluate(prob, words, threads=8, **model), f"{sorted(model)} D={D} v={v}", **model)
    prob, words = batch(D, v, m, times_of_two_words(D, words.shape[2]), n=70)
    copies_same(prob, words, n, oracle.evaluate(prob, words, threads=8), f"times of two words D={D} v={v}")


@pytest.mark.parametrize("D,v,m", [(2, 2, 9), (3, 4, 7), (6, 1, 12), (16, 2, 10)])
def test_lists_without_w_items(D, v, m):
    prob, words = batch(D, v, m, n=70)
    stride = words.shape[2]
    which = np.arange(SPREAD + 300) % len(words)
    ref = oracle.wslide(prob, words, stride, threads=8)
    h = fp.Problem(prob, stride, device=0)
    got = h.wslide(torch.from_numpy(words[which].view(np.int16)).cuda(), stride)
    torch.cuda.synchronize()
    assert_same({name: got[name].cpu().numpy() for name in ("makespan", "idle", "peak", "flags")},
                {name: ref[name][which] for name in ("makespan", "idle", "peak", "flags")}, f"D={D}")
    h.close()


def test_synchronisation():
    rng = np.random.default_rng(29)
    for trial in range(12):
        prob, group, pairs = random_slot_sync_problem(rng)
        lists = lists_of(prob, group, pairs, rng)
        if not lists or (not pairs and max(group) == 1):
            continue
        words = batch_from_lists(lists)
        ref = oracle.evaluate_sync(prob, words, group=group, pairs=pairs)
        which = np.arange(SPREAD + 300) % len(words)
        h = fp.Problem(prob, words.shape[2], device=0)
        h.set_sync(group, pairs)
        res = h.evaluate(torch.from_numpy(words[which].view(np.int16)).cuda())
        assert_same({name: t.cpu().numpy() for name, t in res.items()}, {name: v[which] for name, v in ref.items()}, f"trial {trial}")
        h.close()


@pytest.mark.parametrize("D,v,m", DEVICE_BY_DEVICE)
def test_order_rows_device_by_device_in_one_launch(D, v, m):
    prob, words = order_batch(D, v, m, 40)
    ref = oracle.evaluate(prob, words, threads=8)
    for n in (64, 300, SPREAD):
        copies_same(prob, words, n, ref, f"D={D} v={v} n={n}")
