"""The work a user of this framework has it do, as cases that can be timed.

A case is one pass of a search step through the public entry points: candidate schedules that sit in device
memory are timed and ranked (``evaluate``), parameter sets are turned into schedules, improved, timed and ranked
(``search``), or the tuner's whole grid is run (``tune``).  ``listed`` names the cases, ``draw`` gives more of the
same ranges, ``prepare`` makes what a program has in hand before the call, ``run`` is the call.
"""
from __future__ import annotations

import dataclasses
import random

import numpy as np
import torch

import paper_2510_05112_amd as fp
import workloads
from paper_2510_05112_amd import tuner
from workloads.problem import B, F, FD, L, O, R, W, make_problem

#: What an evaluation case is unless it says otherwise: a chain of `chunks` stages per device, split backward.
_EVALUATE = dict(kind="evaluate", graph="chain", devices=8, microbatches=32, chunks=2, split_backward=True,
                 recompute=False, offload=False, deadlock_per_mille=0, time_scale=1, links=False,
                 microbatch_costs=False, copy_depth=0, candidates=1024, k=16, report="topk")
_SEARCH = dict(kind="search", devices=16, microbatches=64, chunks=2, fused=True, sets=1024, k=16)
_TUNE = dict(kind="tune", devices=8, microbatches=32, chunks=2, k=8)


def listed():
    ev, se, tu = (lambda **x: dict(_EVALUATE, **x)), (lambda **x: dict(_SEARCH, **x)), (lambda **x: dict(_TUNE, **x))
    return [
        # the tuner's grid for one placement of a small job, from Python lists to the best schedules
        tu(name="tune_8x32"),
        # a serving loop that asks for the best of a few small schedules, without a workspace of its own
        ev(name="evaluate_4x8_small", devices=4, microbatches=8, chunks=1, split_backward=False, candidates=1024,
           report="static"),
        # interleaved stages on one node; some candidates deadlock; the alternatives are looked at in several orders
        ev(name="evaluate_8x32", deadlock_per_mille=20, candidates=65536, report="all"),
        # a medium job, a large batch: randomised search over orders
        ev(name="evaluate_16x64", devices=16, microbatches=64, candidates=262144, k=64),
        # the largest job, activations recomputed in part: the batch is several GB
        ev(name="evaluate_32x128_recompute", devices=32, microbatches=128, recompute=True, candidates=65536, k=128),
        # two towers that merge (a multimodal model), activations offloaded in part
        ev(name="evaluate_towers_offload", graph="towers", devices=16, microbatches=64, chunks=1, offload=True,
           deadlock_per_mille=10, candidates=131072, k=64),
        # the same with the transfers beside the computation; sizes that are no powers of two
        ev(name="evaluate_towers_copy_odd", graph="towers", devices=16, microbatches=45, chunks=1, offload=True,
           copy_depth=3, candidates=20011, k=100),
        # micro-batches of unequal length and links that carry one value at a time; an odd machine
        ev(name="evaluate_11x45_links_costs", devices=11, microbatches=45, chunks=3, links=True, microbatch_costs=True,
           candidates=20011, k=100),
        # the towers exchange their states every few micro-batches through a synchronisation instruction
        ev(name="evaluate_sync", graph="sync", devices=12, microbatches=64, chunks=1, candidates=65536, k=64),
        # durations as a profiler hands them out, in microseconds
        ev(name="evaluate_16x64_microseconds", devices=16, microbatches=64, time_scale=1000, candidates=8192, k=64),
        # one step of a search over scheduling priorities at the largest job: generate, slide, time, rank, winners' lists
        se(name="search_32x128_fused", devices=32, microbatches=128, sets=16384, k=128),
        # the same step through lists in memory, which the program keeps
        se(name="search_16x64_lists", fused=False, sets=32768, k=64),
    ]


def _log_int(rng, lo, hi):
    """An integer of lo..hi, spread over its logarithm."""
    return max(lo, min(hi, round(lo * (hi / lo) ** rng.random())))


def draw(rng):
    pick = rng.random()
    if pick < 0.08:
        chunks = rng.choice([1, 2, 2, 3, 4])
        return dict(_TUNE, devices=rng.randint(2, 24), microbatches=_log_int(rng, 4, 96), chunks=chunks,
                    k=rng.randint(1, 32))
    if pick < 0.30:
        c = dict(_SEARCH, devices=rng.randint(2, 32), microbatches=_log_int(rng, 8, 128), chunks=rng.choice([1, 2, 2, 3, 4]),
                 fused=rng.random() < 0.5, k=rng.randint(1, 128))
        items = 3 * c["devices"] * c["microbatches"] * c["chunks"]
        most = min(65536, (400_000_000 if c["fused"] else 200_000_000) // items)
        return dict(c, sets=_log_int(rng, 256, max(257, most)))
    graph = rng.choice(["chain"] * 6 + ["towers", "towers", "sync"])
    c = dict(_EVALUATE, graph=graph, k=rng.randint(1, 128))
    if graph == "chain":
        c.update(devices=rng.randint(2, 40), microbatches=_log_int(rng, 6, 160), chunks=rng.choice([1, 2, 2, 3, 4]),
                 split_backward=rng.random() < 0.85)
        c.update(recompute=c["split_backward"] and rng.random() < 0.3, deadlock_per_mille=rng.choice([0, 0, 10, 20]))
        model = rng.choice(["plain"] * 6 + ["links", "costs", "both", "microseconds"])
        if model == "microseconds":
            c.update(devices=rng.randint(2, 16), microbatches=_log_int(rng, 6, 64), chunks=rng.choice([1, 2]), time_scale=1000)
        elif model != "plain":
            # (costs per micro-batch: within the tables that every combination of the two models takes)
            c.update(devices=rng.randint(2, 16), microbatches=_log_int(rng, 6, 64), recompute=False,
                     links=model in ("links", "both"), microbatch_costs=model in ("costs", "both"))
    else:
        c.update(devices=16 if graph == "towers" else 12, microbatches=_log_int(rng, 8, 64), chunks=1)
        if graph == "towers":
            c.update(offload=True, copy_depth=rng.choice([0, 0, 1, 2, 4, 7]), deadlock_per_mille=rng.choice([0, 10]))
    most = int(min(262144, 1.5e9 // _ops_per_candidate(c)))
    if c["time_scale"] > 1:
        most = min(most, int(5e7 // _ops_per_candidate(c)))
    if c["copy_depth"]:
        most = min(most, 65536)
    c["candidates"] = _log_int(rng, min(256, most), most)
    c["report"] = rng.choice(["topk", "topk", "static", "all"]) if c["candidates"] <= 65536 else "topk"
    return c


# ---- problems ------------------------------------------------------------------------------------------------

def _stages(case):
    # (the synchronisation stage has one item for every four micro-batches)
    return {"towers": 16, "sync": 12.25}.get(case.get("graph"), case["devices"] * case["chunks"])


def _ops_per_candidate(case):
    """Expected number of op words of one candidate."""
    s, m = _stages(case), case["microbatches"]
    ops = s * m * (3 if case.get("split_backward", True) else 2)
    if case.get("recompute"):
        ops *= 1 + 0.219 / 3     # a share of 0, 1/8, 1/4 or 1/2 of the activations is computed twice
    if case.get("offload"):
        ops *= 1 + 0.25 / 3      # a share of 0, 1/8 or 1/4 is moved out and back
    return ops


def _chain(case, seed):
    """A chain with circular placement; costs drawn per stage as in benchmark configuration 4."""
    rng = random.Random(seed)
    p, m, v, scale = case["devices"], case["microbatches"], case["chunks"], case.get("time_scale", 1)
    n = p * v

    def costs(lo, hi):
        return [rng.randint(lo * scale, hi * scale) for _ in range(n)]
    f = costs(20, 30)
    dur = {F: f, B: costs(40, 60), FD: f, R: f}
    split = case.get("split_backward", True)
    if split:
        dur[W] = costs(15, 25)
    comm = costs(2, 6)
    return make_problem(p, n, m, int(split), [s % p for s in range(n)], [(s, s + 1, comm[s]) for s in range(n - 1)],
                        dur, mem_cap=max(3, 3 * p // 4))


def _candidates(case, seed, device):
    """(problem, op words on the GPU, synchronisation groups, pairs): seeded list schedules; the batch is filled with
    copies of them in which weight-gradient items are delayed here and there, a search's neighbourhood move that is
    always valid (nothing waits for such an item)."""
    n, m, graph = case["candidates"], case["microbatches"], case["graph"]
    n_base = min(n, 2048, max(96, int(1.0e8 // (_ops_per_candidate(case) * case["devices"]))))
    group = pairs = None
    if graph == "sync":
        spec = workloads.sync_config(n_base)
        prob = spec.problem
        if m != prob.n_microbatches:
            prob = dataclasses.replace(prob, n_microbatches=m)
        longest = 3 * m + 3 * (-(-m // int(spec.group[-1])))
        spec = dataclasses.replace(spec, problem=prob, seed=seed, stride=-(-longest // 8) * 8)
        group, pairs = spec.group, spec.pairs
        words = workloads.generate_sync(spec)
    else:
        if graph == "towers":
            prob = dataclasses.replace(workloads.config(5, n_base).problem, n_microbatches=m)
            cap = 12
        else:
            prob = _chain(case, seed)
            cap = int(prob.mem_cap[0])
        rows = m * case["chunks"] * (3 if case["split_backward"] else 2)
        marks = max(1, m * case["chunks"] // 2)
        longest = rows + (marks if case["recompute"] else 0) + (2 * marks if case["offload"] else 0)
        spec = workloads.Spec(0, prob, n_base, -(-longest // 8) * 8, case["k"], recompute=int(case["recompute"]),
                              offload=int(case["offload"]), max_marks_per_device=marks, cap_units=cap, seed=seed,
                              deadlock_per_mille=case["deadlock_per_mille"])
        words = workloads.generate(spec)
    base = torch.from_numpy(words.view(np.int16)).to(device)
    gen = torch.Generator(device=device).manual_seed(seed)
    which = torch.randint(n_base, (n,), device=device, generator=gen)
    which[:n_base] = torch.arange(n_base, device=device)
    ops = torch.empty((n,) + tuple(base.shape[1:]), dtype=torch.int16, device=device)
    step = max(1, (1 << 27) // base[0].numel())
    for lo in range(0, n, step):
        part = base.index_select(0, which[lo:lo + step]).unflatten(2, (-1, 2))
        kind = (part >> 13) & 7
        move = (kind[..., 0] == W) & (kind[..., 1] != 0)
        move &= torch.randint(8, move.shape, dtype=torch.uint8, device=device, generator=gen) == 0
        ops[lo:lo + step] = torch.where(move.unsqueeze(-1), part.flip(-1), part).flatten(2)
    return prob, ops, group, pairs


def prepare(case, seed):
    device = torch.device("cuda", torch.cuda.current_device())
    if case["kind"] == "tune":
        prob = _chain(case, seed)
        return dict(kind="tune", problem=prob, k=case["k"], circular=case["chunks"] > 1,
                    handle=fp.Problem(prob, tuner.stride_for(prob), device=device.index))
    k = case["k"]
    top = dict(idx=torch.empty(k, dtype=torch.int64, device=device), makespan=torch.empty(k, dtype=torch.int64, device=device),
               count=torch.empty(1, dtype=torch.int32, device=device))
    if case["kind"] == "search":
        prob = _chain(case, seed)
        n, stride = case["sets"], tuner.stride_for(prob)
        handle = fp.Problem(prob, stride, device=device.index)
        policy, inflight = workloads.policy_sets(prob, n, seed)
        lists = k if case["fused"] else n
        state = dict(kind="search", fused=case["fused"], handle=handle, stride=stride, k=k, top=top,
                     policy=torch.from_numpy(policy).to(device), inflight=torch.from_numpy(inflight).to(device),
                     results=handle.alloc_results(n), workspace=handle.alloc_workspace(n, k),
                     lists=dict(ops=torch.empty((lists, prob.n_devices, stride), dtype=torch.int16, device=device),
                                steps=torch.empty(lists, dtype=torch.int32, device=device),
                                status=torch.empty(lists, dtype=torch.uint8, device=device)),
                     steps=dict(steps=torch.empty(n, dtype=torch.int32, device=device),
                                status=torch.empty(n, dtype=torch.uint8, device=device)))
        slide_bytes = int(fp.load_library().fpsched_wslide_workspace_bytes(handle._h, lists, stride))
        state["slide_workspace"] = torch.empty(slide_bytes, dtype=torch.uint8, device=device)
        state["slid"] = dict(ops=torch.empty_like(state["lists"]["ops"]), **handle.alloc_results(lists))
        return state
    prob, ops, group, pairs = _candidates(case, seed, device)
    handle = fp.Problem(prob, ops.shape[2], device=device.index)
    if case["links"]:
        handle.set_link_occupancy(True)
    if case["microbatch_costs"]:
        handle.set_microbatch_costs(workloads.microbatch_costs(prob, seed))
    if case["copy_depth"]:
        handle.set_copy_engine(case["copy_depth"])
    if group is not None:
        handle.set_sync(group, pairs)
    n = case["candidates"]
    return dict(kind="evaluate", report=case["report"], handle=handle, ops=ops, k=k, top=top,
                results=handle.alloc_results(n), workspace=handle.alloc_workspace(n, k))


def run(state):
    handle, k = state["handle"], state["k"]
    if state["kind"] == "tune":
        best = tuner.tune(handle, state["problem"], state["circular"], k=k, slide=True)
        return {name: np.asarray([int(b[name]) for b in best], np.int64) for name in ("makespan", "index", "slid")}
    results, top, workspace = state["results"], state["top"], state.get("workspace")
    if state["kind"] == "evaluate":
        if state["report"] == "static":
            handle.evaluate_topk_static(state["ops"], k, results, top)
            return dict(results=results, top=top)
        handle.evaluate(state["ops"], results, workspace)
        handle.topk(results, k, workspace, top)
        if state["report"] == "all":
            return dict(results=results, top=top, rank=handle.rank(results, k), front=handle.pareto(results, 256))
        return dict(results=results, top=top)
    policy, inflight, lists = state["policy"], state["inflight"], state["lists"]
    if state["fused"]:
        handle.generate_evaluate(policy, inflight, results=results, out=state["steps"], workspace=workspace, slide=True)
        handle.topk(results, k, workspace, top)
        handle.generate_selected(policy, inflight, top["idx"], state["stride"], out=lists, workspace=workspace)
        slid = handle.wslide(lists["ops"], state["stride"], out=state["slid"], workspace=state["slide_workspace"])
        return dict(results=results, steps=state["steps"], top=top, winners=slid)
    handle.generate(policy, inflight, state["stride"], out=lists, workspace=workspace)
    slid = handle.wslide(lists["ops"], state["stride"], out=state["slid"], workspace=state["slide_workspace"])
    handle.topk(slid, k, workspace, top)
    return dict(lists=lists, slid=slid, top=top)


def work(case):
    """Op words in or out once, results out once; an op costs a comparison of two times and two additions, and one
    addition and one comparison for its memory."""
    devices, m = case["devices"], case["microbatches"]
    results = 8 + 12 * devices + 1
    if case["kind"] == "evaluate":
        ops = case["candidates"] * _ops_per_candidate(case)
        return {"bytes": 2 * ops + case["candidates"] * results, "flops": 5 * ops}
    sets = case["sets"] if case["kind"] == "search" else 32 * (2 if case["chunks"] > 1 else 1)
    ops = 3.0 * sets * _stages(case) * m
    inputs = sets * (32 * devices + 4 * _stages(case))
    if case["kind"] == "search" and not case["fused"]:
        # the generated lists and the improved ones are what the program keeps
        return {"bytes": inputs + 4 * ops + sets * (results + 5), "flops": 10 * ops}
    return {"bytes": inputs + sets * (results + 5), "flops": 10 * ops}


def tolerance(case):
    """Every result is a whole number."""
    return "exact"
