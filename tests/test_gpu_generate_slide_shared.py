"""The sliding form of the generator with as many sets in a wavefront as a large batch has (more than two for each SIMD): graphs
with two inputs or outputs per stage, stashes deeper than a queue word, and how its segments come by their sets.  The batches are
copies of a few sets, so that the oracles have these only to do.  (That they are launched so: test_host_launches.py.)"""
import copy

import numpy as np
import pytest
import torch

import oracle
import paper_2510_05112_amd as fp
from helpers import dag_problem, two_tower_problem
from test_genoracle import random_policies, stride_for
from test_gpu_generate_evaluate import placed_chain

pytestmark = pytest.mark.gpu

FULL = 2 * 4 * 256 + 77   # more than two sets for each SIMD of 256 compute units


def fork_and_join(per_device, n_devices, m):
    # (0, 1) -> 2 -> (3, 4) -> 5, twice with eight stages and more
    n = per_device * n_devices
    edges = [(0, 2), (1, 2), (2, 3), (2, 4), (3, 5), (4, 5)] + [(s - 1, s) for s in range(6, n)]
    return dag_problem(edges, n, [s % n_devices for s in range(n)], n_devices, m=m, has_w=1, seed=n + n_devices)


def graphs():
    yield "two towers", two_tower_problem(m=5, has_w=1, comm=2)
    yield "fork and join, one stage per device", fork_and_join(1, 6, 7)
    yield "fork and join, two", fork_and_join(2, 3, 6)
    yield "fork and join, four", fork_and_join(4, 2, 5)
    yield "round two devices", placed_chain(2, 2, 9, 1, seed=3)
    yield "up and down", placed_chain(4, 2, 6, 1, seed=4, circular=False)


def deep_stashes():
    for D in (2, 3):
        for v, m in ((2, 48), (4, 20), (1, 70)):
            base = placed_chain(D, v, m, 1, seed=40 + v)
            S = D * v
            for name, costs in (("none fits", [5000] * S), ("some fit", ([1, 300] * S)[:S]), ("any", list(np.random.default_rng(S).integers(0, 60, S))), ("no cost", [0] * S)):
                prob = copy.deepcopy(base)
                prob.dur[3] = costs
                yield f"{D} x {m} x {v}, {name}", prob


# with one wavefront for each of 256 compute units, devices, stages per device, micro-batches, sets, sets per wavefront, classes (0: a segment to each set)
ORDERS = ((20, 2, 3, 300, 1, 1), (20, 2, 3, 320, 1, 4), (20, 2, 3, 1459, 2, 4), (20, 2, 3, 2100, 3, 4), (20, 2, 2, 1459, 2, 4), (20, 2, 2, 2100, 3, 1),
          (7, 3, 5, 2100, 9, 0), (7, 3, 5, 6000, 9, 4), (7, 3, 4, 6000, 9, 1))


def check_copies(prob, n, what, distinct=70):
    rng = np.random.default_rng(prob.n_devices * 100 + prob.n_stages)
    pol, inf = random_policies(rng, distinct, prob, rng.random(distinct) < 0.5)
    st = stride_for(prob)
    gen = oracle.generate(prob, pol, inf, st, threads=8)
    ref = oracle.wslide(prob, gen["words"], st, threads=8)
    which = np.arange(n) % distinct
    h = fp.Problem(prob, st, device=0)
    res, out = h.generate_evaluate(torch.from_numpy(np.ascontiguousarray(pol[which], np.int32)).cuda(),
                                   torch.from_numpy(np.ascontiguousarray(inf[which], np.int32)).cuda(), slide=True)
    torch.cuda.synchronize()
    got = {**{k: v.cpu().numpy() for k, v in res.items()}, "steps": out["steps"].cpu().numpy(), "status": out["status"].cpu().numpy()}
    h.close()
    for name, want in (("status", gen["status"]), ("steps", gen["steps"]), ("flags", ref["flags"]), ("makespan", ref["makespan"]),
                       ("idle", ref["idle"]), ("peak", ref["peak"])):
        bad = np.flatnonzero((got[name] != want[which]).reshape(n, -1).any(1))
        assert not len(bad), f"{what}: {name} differs for {len(bad)} sets, first {bad[:5]}"


@pytest.mark.parametrize("name,prob", [pytest.param(*p, id=p[0].replace(" ", "_")) for p in graphs()])
def test_several_sets_in_a_wavefront(name, prob):
    check_copies(prob, FULL, name)


@pytest.mark.parametrize("name,prob", [pytest.param(*p, id=p[0].replace(" ", "_")) for p in deep_stashes()])
def test_deep_stashes_of_several_sets(name, prob):
    check_copies(prob, FULL, name, distinct=60)


@pytest.mark.parametrize("D,v,m,n,per_wave,classes", ORDERS)
def test_orders(D, v, m, n, per_wave, classes, monkeypatch):
    monkeypatch.setenv("FPSCHED_GEN_WAVES", "1")
    check_copies(placed_chain(D, v, m, 1, seed=D), n, f"{n} sets", distinct=150)
