"""The two forms of the synchronisation model that count as the slot kernel: the two-pass evaluation's, and the
one-kernel form for settings in which an op has more than two edge slots (and wherever FPSCHED_SYNC_SLOTS asks for it).
What fpsched_problem_set_sync prints says which one a setting got."""
import numpy as np
import pytest

import oracle
import workloads
from gpu_common import assert_same
from helpers import batch_from_lists, perturb, random_slot_sync_problem, random_sync_lists
from workloads.problem import B, F, W, make_problem, pack_word

pytestmark = pytest.mark.gpu

TWO_PASS, ONE_KERNEL = "[fpsched] list evaluation, synchronisation", "[fpsched] slot kernel, synchronisation"


def evaluate(prob, words, group, pairs, capfd):
    """(results, the form that was chosen)"""
    import torch
    import paper_2510_05112_amd as fp
    h = fp.Problem(prob, words.shape[2], device=0)
    capfd.readouterr()
    h.set_sync(group, pairs)
    said = capfd.readouterr().err
    assert (TWO_PASS in said) != (ONE_KERNEL in said), said
    assert h.active_kernel() == "slots"
    res = h.evaluate(torch.from_numpy(words.view(np.int16)).cuda())
    out = {name: t.cpu().numpy() for name, t in res.items()}
    h.close()
    return out, TWO_PASS if TWO_PASS in said else ONE_KERNEL


def lists_of(prob, group, pairs, rng):
    lists = []
    for t in range(6):
        base = random_sync_lists(prob, group, pairs, rng, 0.25 * (t % 2), 0.25 * ((t // 2) % 2))
        if base is not None:
            lists += [base, perturb(base, rng, 1 + t % 3)]
    return lists


@pytest.mark.parametrize("form", [TWO_PASS, ONE_KERNEL])
def test_settings_that_both_forms_take(form, monkeypatch, capfd):
    monkeypatch.setenv("FPSCHED_VERBOSE", "1")
    if form == ONE_KERNEL:
        monkeypatch.setenv("FPSCHED_SYNC_SLOTS", "1")
    rng = np.random.default_rng(17)
    forms, n_grouped, n_dead = [], 0, 0
    for trial in range(30):
        prob, group, pairs = random_slot_sync_problem(rng)
        lists = lists_of(prob, group, pairs, rng)
        if not lists or (not pairs and max(group) == 1):   # (nothing to switch on)
            continue
        words = batch_from_lists(lists)
        words[-1, 0, 0] = pack_word(F, 0, 2047)   # an item index beyond its stage's item count
        ref = oracle.evaluate_sync(prob, words, group=group, pairs=pairs)
        out, chosen = evaluate(prob, words, group, pairs, capfd)
        assert_same(out, ref, f"trial {trial} {chosen}")
        forms.append(chosen)
        n_grouped += any(g > 1 for g in group)
        n_dead += int((ref["flags"] & 1).sum())
    assert forms.count(form) > (20 if form == TWO_PASS else len(forms) - 1) and n_grouped > 10 and n_dead > 15


@pytest.mark.parametrize("form", [TWO_PASS, ONE_KERNEL])
def test_the_multimodal_workload(form, monkeypatch, capfd):
    monkeypatch.setenv("FPSCHED_VERBOSE", "1")
    if form == ONE_KERNEL:
        monkeypatch.setenv("FPSCHED_SYNC_SLOTS", "1")
    spec = workloads.sync_config(700)
    words = workloads.generate_sync(spec, threads=8)
    out, chosen = evaluate(spec.problem, words, spec.group, spec.pairs, capfd)
    assert chosen == form
    assert_same(out, oracle.evaluate_sync(spec.problem, words, spec.group, spec.pairs, threads=8), form)


@pytest.mark.parametrize("m,grouped", [(1, False), (9, False), (40, False), (40, True)])
def test_a_stage_with_three_edge_slots_gets_the_one_kernel_form(m, grouped, monkeypatch, capfd):
    # stage 2 of a chain takes in and gives away a pair's value: its two inputs and its two outputs are of three classes
    monkeypatch.setenv("FPSCHED_VERBOSE", "1")
    rng = np.random.default_rng(m)
    S = 6
    dur = {F: rng.integers(1, 9, S), B: rng.integers(1, 9, S), W: rng.integers(0, 5, S)}
    prob = make_problem(S, S, m, 1, list(range(S)), [(s, s + 1, 1 + s % 3) for s in range(S - 1)], dur, mem_cap=4 * m)
    group, pairs = [1] * S, [(F, 0, F, 2, 4), (F, 2, F, 4, 1)]
    if grouped:
        group[5] = 7
    lists = lists_of(prob, group, pairs, rng)
    assert lists
    words = batch_from_lists(lists)
    ref = oracle.evaluate_sync(prob, words, group=group, pairs=pairs)
    out, chosen = evaluate(prob, words, group, pairs, capfd)
    assert chosen == ONE_KERNEL and (ref["flags"] == 0).any()
    assert_same(out, ref, f"m {m}")


@pytest.mark.parametrize("every", [2, 3, 4, 5, 9, 64])
@pytest.mark.parametrize("m", [8, 33, 64])
def test_groups_of_all_sizes_and_remainders(every, m, capfd, monkeypatch):
    """Groups below, at and above the values taken in at a time, with whole and partial last groups, and a device whose list
    has one such item behind the other; more candidates than a launch has segments."""
    import dataclasses
    monkeypatch.setenv("FPSCHED_VERBOSE", "1")
    spec = workloads.sync_config(300, every)
    prob = dataclasses.replace(spec.problem, n_microbatches=m)
    longest = 3 * m + 3 * (-(-m // every))
    spec = dataclasses.replace(spec, problem=prob, group=np.minimum(spec.group, m), stride=-(-longest // 8) * 8, swap_per_mille=60)
    words = np.tile(workloads.generate_sync(spec, threads=4), (60 if (every, m) == (4, 64) else 1, 1, 1))
    out, form = evaluate(prob, words, spec.group, spec.pairs, capfd)
    assert form == TWO_PASS
    assert_same(out, oracle.evaluate_sync(prob, words, spec.group, spec.pairs, threads=8), f"{every} of {m}")
