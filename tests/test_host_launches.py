"""Which kernels a call launches, without a GPU: every test runs in a process of its own in which a stand-in for the HIP runtime
(hip_stub.c) comes before the real one, so that launches are only noted."""
import ctypes
import os
import pickle
import re
import shutil
import subprocess
import sys

import numpy as np
import pytest

import paper_2510_05112_amd as fp
import workloads
from helpers import two_tower_problem
from workloads.problem import F, L, O, chain_problem

HERE = os.path.dirname(os.path.abspath(__file__))
HEADERS = "/opt/rocm/include"
pytestmark = pytest.mark.skipif(not (shutil.which("gcc") and os.path.isdir(os.path.join(HEADERS, "hip"))), reason="no compiler, no HIP headers")


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    path = str(tmp_path_factory.mktemp("stub") / "hip_stub.so")
    subprocess.run(["gcc", "-shared", "-fPIC", "-O1", "-I" + HEADERS, "-o", path, os.path.join(HERE, "hip_stub.c")], check=True)
    return path


def run(stub, what, *args):
    """Runs the function `what` of this file in a new process, with the stand-in (and without torch, which brings the runtime)."""
    code = (f"import pickle, sys; sys.path[:0] = [{HERE!r}, {os.path.dirname(HERE)!r}]; import test_host_launches as t; "
            f"t.{what}(t.Device({stub!r}), *pickle.loads(sys.stdin.buffer.read()))")
    done = subprocess.run([sys.executable, "-c", code], input=pickle.dumps(args), stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    assert done.returncode == 0, done.stdout.decode()


class Device:
    """In the new process: the stand-in, and calls with pointers that nothing looks at."""

    def __init__(self, stub):
        self.stub = ctypes.CDLL(stub, mode=ctypes.RTLD_GLOBAL)
        self.stub.stub_launched.restype = ctypes.c_char_p
        self.lib = fp.load_library()
        self.results = fp.binding._Results(4096, 4096, 4096, 4096)

    def launched(self, rc=0, what=0):
        assert rc == what, rc
        names = [self.stub.stub_launched(i).decode() for i in range(self.stub.stub_launches())]
        self.forms = [tuple(int(x) for x in re.findall(r"L[bi](\d+)E", n)) for n in names]   # (template arguments)
        self.waves = [self.stub.stub_grid(i) * self.stub.stub_block(i) // 64 for i in range(len(names))]
        self.shapes = [(self.stub.stub_grid(i), self.stub.stub_block(i)) for i in range(len(names))]
        self.lds = [self.stub.stub_lds(i) for i in range(len(names))]
        self.words = [self.stub.stub_word(i) & 0xffffffff for i in range(len(names))]
        self.stub.stub_reset()
        return [re.search(r"\d([a-z_]+_kernel)", n).group(1) for n in names]

    def evaluate(self, h, stride, n=1, what=0):
        return self.launched(self.lib.fpsched_evaluate(h._h, 4096, n, stride, self.results, 4096, 1 << 20, None), what)

    def wslide(self, h, stride, n=1, stride_out=64):
        size = self.lib.fpsched_wslide_workspace_bytes(h._h, n, stride)
        return self.launched(self.lib.fpsched_wslide(h._h, 4096, n, stride, 4096, stride_out, self.results, 4096, size, None))

    def copy_form(self, h, stride, n):
        """What the copy engine is timed by: "one kernel", or the transfers that the two passes keep."""
        got = self.evaluate(h, stride, n)
        if got == ["reset_counter_kernel", "eval_slot_kernel"]:
            return "one kernel"
        assert got[-2:] == TWO_PASSES
        return self.forms[-1][-1]

    def one_turn(self, h, stride):
        """The largest batch that the one kernel takes (on a problem that goes to it up to a full chip)."""
        least, beyond = 1, 1 << 24
        assert self.copy_form(h, stride, least) == "one kernel" != self.copy_form(h, stride, beyond)
        while beyond - least > 1:
            n = (least + beyond) // 2
            least, beyond = (n, beyond) if self.copy_form(h, stride, n) == "one kernel" else (least, n)
        self.copy_form(h, stride, least)
        assert self.waves[-1] % 256 == 0 and least % self.waves[-1] == 0   # (every wavefront of every compute unit has its candidates)
        return least


LONGEST = (1 << 23) - 32   # rows that the timing pass has positions for
TWO_PASSES = ["check_rows_kernel", "time_lists_kernel"]
KEPT = {1: 3, 2: 3, 3: 3, 4: 4, 5: 7, 6: 7, 7: 7}   # copy engine: transfers that the two passes keep at each depth


def long_rows(dev):
    # times beyond 24 bits: positions of a row of 2^25 words would wrap
    h = fp.Problem(chain_problem(2, 8, v=2, f=2, b=4, w=1, comm=1), 1 << 25, device=0)
    for stride in (64, LONGEST):
        assert dev.evaluate(h, stride) == TWO_PASSES
    for stride in (LONGEST + 8, 1 << 23, 1 << 25):
        assert dev.evaluate(h, stride) == ["eval_general_kernel"]
    h.close()
    # every form with times of 24 bits (a single device, costs of one)
    prob = chain_problem(1, 16, v=2, f=1, b=1, w=1)
    prob.dur[O], prob.dur[L] = 1, 1
    ones = np.ones((8, prob.n_stages, prob.n_microbatches), np.int32)
    forms = {"plain": (lambda h: None, "eval_general_kernel"),
             "costs": (lambda h: h.set_microbatch_costs(ones), "eval_general_kernel"),
             "links": (lambda h: h.set_link_occupancy(True), "eval_general_kernel"),
             "both": (lambda h: (h.set_microbatch_costs(ones), h.set_link_occupancy(True)), "eval_general_kernel"),
             "groups": (lambda h: h.set_sync([2, 1]), "eval_sync_kernel"),
             "pairs": (lambda h: h.set_sync(None, [(F, 1, F, 0, 0)]), "eval_sync_kernel"),
             "copy": (lambda h: h.set_copy_engine(3), "eval_slot_kernel")}
    n = 1 << 20   # (more than the one kernel of the copy engine has side by side)
    for name, (set_model, beyond) in forms.items():
        h = fp.Problem(prob, 1 << 23, device=0)
        set_model(h)
        got = dev.evaluate(h, LONGEST, n)
        assert got[-2:] == TWO_PASSES, (name, got)
        got = dev.evaluate(h, LONGEST + 8, n)
        assert got[-1] == beyond, (name, got)
        h.close()
    h = fp.Problem(prob, 1 << 23, device=0)
    assert dev.wslide(h, LONGEST)[:2] == TWO_PASSES
    assert "eval_slot_kernel" in dev.wslide(h, LONGEST + 8)
    h.close()
    # whole finish-time tables that do not fit LDS: refused
    h = fp.Problem(chain_problem(4, 1500, v=4, f=0, b=0), 1 << 25, device=0)
    assert dev.evaluate(h, LONGEST) == TWO_PASSES
    assert dev.evaluate(h, LONGEST + 8, what=-6) == []
    h.close()


def test_rows_beyond_the_positions_of_the_timing_pass(stub):
    run(stub, "long_rows")


def no_memory_for_copy_tables(dev):
    prob = chain_problem(8, 16, v=2, f=3, b=4, w=2, comm=1)
    prob.dur[O], prob.dur[L] = 2, 2
    for there, depth in ((4, 3), (7, 2), (3, 4), (1, 7)):   # (engines of more than three transfers have tables of their own)
        h = fp.Problem(prob, 128, device=0)
        h.set_copy_engine(there)
        dev.stub.stub_fail_malloc(1)
        h.set_copy_engine(depth)
        assert dev.stub.stub_fail_malloc(0) == 0
        assert dev.copy_form(h, 128, 1 << 16) == "one kernel"
        h.set_copy_engine(depth)
        assert dev.copy_form(h, 128, 1 << 16) == KEPT[depth]
        h.set_copy_engine(there)
        assert dev.copy_form(h, 128, 1 << 16) == KEPT[there]
        h.close()


def no_memory_for_some_table(dev):
    prob = chain_problem(4, 8, v=2, f=3, b=4, w=2, comm=1)
    nth, first = 0, set()
    while True:
        nth += 1
        dev.stub.stub_fail_malloc(nth)
        try:
            h = fp.Problem(prob, 64, device=0)
        except fp.FpschedError as e:
            assert e.code in (-2, -3)
            dev.stub.hipGetLastError()
            continue
        left = dev.stub.stub_fail_malloc(0)
        assert dev.evaluate(h, 64) == TWO_PASSES   # (and no error of the handle's making is reported)
        size = dev.lib.fpsched_wslide_workspace_bytes(h._h, 1, 64)
        rc = dev.lib.fpsched_wslide(h._h, 4096, 1, 64, 4096, 64, dev.results, 4096, size, None)
        if rc == 0:
            first.add(dev.launched()[0])
        else:
            assert dev.launched(rc, -6) == []
        h.close()
        if left > 0:
            break
    assert first == {"check_rows_kernel", "reset_counter_kernel"}   # (the two passes, and the slot kernel without their tables)


@pytest.mark.parametrize("what", ["no_memory_for_copy_tables", "no_memory_for_some_table"])
def test_no_memory_for_a_faster_form(what, stub):
    run(stub, what)


DRAW_SHARE = 10   # (its place among the timing pass's arguments)


def share_of_a_draw(dev):
    dev.stub.stub_watch(b"time_lists_kernel", DRAW_SHARE)

    def share(prob, stride, set_model=lambda h: None, n=1 << 17):
        h = fp.Problem(prob, stride, device=0)
        set_model(h)
        assert dev.evaluate(h, stride, n)[-2:] == TWO_PASSES
        h.close()
        got = dev.words[-1] * dev.waves[-1] / 2**32   # (of a wavefront, rounded up)
        return round(got, 3) if got < 1 else got

    def links(h):
        h.set_link_occupancy(True)
    chain = chain_problem(8, 64, v=2, f=3, b=4, w=2, comm=1)
    towers = workloads.config(5, 1).problem

    def with_costs(prob):
        return lambda h: h.set_microbatch_costs(workloads.microbatch_costs(prob))
    both = {name: (lambda h, prob=prob: (with_costs(prob)(h), links(h))) for name, prob in (("chain", chain), ("towers", towers))}
    assert share(chain, 384) == share(chain, 384, with_costs(chain)) == 0.5
    assert share(chain, 384, links) == share(chain, 384, both["chain"]) == 0.25
    assert share(towers, 256) == share(towers, 256, links) == share(towers, 256, both["towers"]) == 0.5
    assert [share(chain, stride, links) for stride in (184, 192)] == [0.5, 0.25]
    # the longest candidates that more than one of are drawn at a time
    assert (share(chain, 2048), share(chain, 2056)) == (0.5, 0)
    assert (share(chain, 2048, links), share(chain, 2056, links)) == (0.25, 0)


def test_share_of_a_draw(stub):
    run(stub, "share_of_a_draw")


def placement_by_rows(dev):
    def placed_by(D, m, v, rows):
        prob = chain_problem(D, m, v=v, f=2, b=3, w=1, comm=1)
        stride = -(-3 * m * v // 8) * 8
        h = fp.Problem(prob, stride, device=0)
        got = dev.wslide(h, stride, rows // D, stride)
        h.close()
        assert got[-3:-1] == TWO_PASSES
        return {"wslide_place_rows_kernel": "wavefront", "wslide_place_kernel": "lane"}[got[-1]]
    # a row's items: up to 127, up to 447, 448 and more, and the devices
    for shape, most in (((4, 4, 1), 16384), ((5, 4, 1), 12288), ((8, 42, 1), 12288), ((8, 43, 1), 16384), ((9, 43, 1), 12288), ((4, 74, 2), 16384),
                        ((8, 149, 1), 16384), ((16, 64, 2), 12288), ((32, 149, 1), 12288), ((16, 75, 2), 24576), ((4, 75, 2), 24576), ((32, 128, 2), 24576)):
        D = shape[0]
        assert placed_by(*shape, most // D * D) == "wavefront", shape
        assert placed_by(*shape, most // D * D + D) == "lane", shape


def test_placement_by_rows(stub):
    run(stub, "placement_by_rows")


def copy_rule(dev):
    def engine(prob, depth, stride=256):
        prob.dur[O], prob.dur[L] = 2, 3
        h = fp.Problem(prob, stride, device=0)
        h.set_copy_engine(depth)
        return h

    def chain(D, m, v=1, has_w=1):
        return chain_problem(D, m, v=v, f=3, b=4, w=2 if has_w else None, comm=1)
    # more than one turn of the one kernel, whatever the problem; one turn of two devices
    for depth in KEPT:
        for prob in (chain(2, 6, 2), chain(1, 40), chain(2, 40, 4)):
            h = engine(prob, depth, 640)
            most = dev.one_turn(h, 640)
            assert [dev.copy_form(h, 640, n) for n in (1, most, most + 1)] == ["one kernel", "one kernel", KEPT[depth]]
            h.close()
    # one turn of more devices: the forms of each side of a row's items, the second edges, the depth and the stages per device
    towers = [two_tower_problem(m=m, has_w=has_w, comm=2, mem_cap=3) for m, has_w in ((21, 1), (31, 0), (22, 1), (32, 0))]
    for depth, prob, form in [(3, chain(3, 2), 3), (1, chain(40, 2), 3),
                              (1, towers[0], "one kernel"), (3, towers[1], "one kernel"), (1, towers[2], 3), (3, towers[3], 3),
                              (4, chain(3, 31), "one kernel"), (4, chain(3, 32), 4), (4, chain(3, 47, 1, 0), "one kernel"), (4, chain(3, 48, 1, 0), 4),
                              (4, towers[2], "one kernel"),
                              (5, chain(3, 32), "one kernel"), (7, chain(9, 80), "one kernel"), (5, chain(3, 16, 2), 7), (7, chain(3, 15, 2), "one kernel")]:
        h = engine(prob, depth)
        assert dev.copy_form(h, 256, 1) == form, (prob.name, depth)
        if form == "one kernel":
            most = dev.one_turn(h, 256)
            assert dev.copy_form(h, 256, most + 1) == KEPT[depth]
        else:
            assert dev.copy_form(h, 256, 1 << 22) == form
        h.close()


def test_copy_engine_forms(stub):
    run(stub, "copy_rule")


def copy_forms_of(dev, problems, depth, lists, want):
    seen = set()
    for prob in problems:
        h = fp.Problem(prob, 256, device=0)
        h.set_copy_engine(depth)
        seen.add(dev.copy_form(h, 256, lists))
        # (a copy more than fills the chip goes to the two passes: copy_rule)
        assert dev.copy_form(h, 256, 1 << 22) == want[-1]
        h.close()
    assert seen == set(want), seen


@pytest.mark.parametrize("depth", [1, 2, 3, 4, 5, 7])
def test_forms_that_the_tests_of_the_copy_engine_run(depth, stub):
    import test_gpu_copy
    import test_gpu_copy_deep
    if depth <= 4:
        run(stub, "copy_forms_of", test_gpu_copy.form_problems(), depth, test_gpu_copy.FORM_LISTS, ["one kernel", KEPT[depth]])
    if depth in test_gpu_copy_deep.DEPTHS:
        run(stub, "copy_forms_of", test_gpu_copy_deep.form_problems(), depth, test_gpu_copy.FORM_LISTS, ["one kernel", KEPT[depth]])


def rows_shared(dev, evaluated, without_w, drawn):
    SHARED = 2   # (of the order pass's template arguments)

    def order_pass(prob, stride, rows):
        h = fp.Problem(prob, stride, device=0)
        got = dev.evaluate(h, stride, -(-rows // prob.n_devices))
        h.close()
        assert got[-2:] == TWO_PASSES
        return dev.forms[-2][SHARED], "reset_counter_kernel" in got
    for prob, stride, rows in evaluated:
        assert order_pass(prob, stride, rows) == (1, False)
    for prob, stride, rows in without_w:
        h = fp.Problem(prob, stride, device=0)
        assert dev.wslide(h, stride, -(-rows // prob.n_devices), stride)[:2] == TWO_PASSES
        h.close()
        assert dev.forms[0][1:] == (1, 1)
    assert order_pass(*drawn) == (1, True)
    # either side of the lines: eight wavefronts of rows per compute unit, rows of 64 words, wavefronts that the states leave room for
    one, stride = chain_problem(1, 24, v=1, f=3, b=5, w=2, comm=1), 72
    assert [order_pass(one, stride, 64 * 2048 + more)[0] for more in (0, 1)] == [0, 1]
    assert [order_pass(one, stride, 1 << 20)[0] for stride in (56, 64, 72)] == [0, 1, 1]
    assert [order_pass(chain_problem(32, m, v=2, f=3, b=5, w=2, comm=1), 768, 1 << 20)[0] for m in (64, 128)] == [1, 0]


def test_rows_that_four_lanes_share(stub):
    import test_gpu_rows_shared as t
    run(stub, "rows_shared", [(*t.problem_of(*case[:3], padding), case[3]) for case in t.EVALUATED for padding in t.PADDINGS],
        [(*t.problem_of(*case[:3], 8), case[3]) for case in t.WITHOUT_W], (*t.problem_of(*t.DRAWN[:3], 8), t.DRAWN[3]))


def draws(dev, cases):
    LEAST = 9   # (its place among the timing pass's arguments)
    for prob, stride, waves, least, most, factors in cases:
        h = fp.Problem(prob, stride, device=0)
        cpw = h.info()["candidates_per_wave"]
        segments = 256 * waves * cpw
        word = {}
        for argument in (LEAST, DRAW_SHARE):
            dev.stub.stub_watch(b"time_lists_kernel", argument)
            dev.evaluate(h, stride, segments + 1)
            assert dev.waves[-1] == 256 * waves
            word[argument] = dev.words[-1]
        h.close()
        # a wavefront's first draw of the largest batch
        left = int(segments * max(factors)) - segments
        assert word[LEAST] == least and max(least, min(left * word[DRAW_SHARE] >> 32, cpw)) == most


def test_draws(stub):
    import test_gpu_draws as t
    run(stub, "draws", [(*t.problem_of(*case[:3]), *case[3:]) for case in t.CASES])


def generator_forms(dev, problems):
    ONE_NEIGHBOUR = 3   # (of the template arguments, the second)
    for name, prob, want in problems:
        h = fp.Problem(prob, 256, device=0)
        dev.launched(dev.lib.fpsched_generate(h._h, 4096, 4096, 100, 256, 4096, 4096, 4096, 4096, 1 << 20, None))
        h.close()
        assert (dev.forms[-1][1] == ONE_NEIGHBOUR) == want, name


def test_generator_forms(stub):
    import test_gpu_generate_neighbours as t
    run(stub, "generator_forms", [(name, prob, not name.startswith(("up and down", "three stages", "two stages", "forward"))) for name, prob in t.problems()])


def small_batches_of_variants(dev, problems):
    # up to four candidates for each of 256 compute units: one to a wavefront, or where up to six devices have four stages all of a
    # compute unit's; one workgroup to a compute unit, however many workgroups a large batch has there
    groups = set()
    for prob, set_model in problems:
        stride = -(-3 * prob.n_microbatches * 4 // 8) * 8 + 8
        h = fp.Problem(prob, stride, device=0)
        if set_model == "costs":
            h.set_microbatch_costs(workloads.microbatch_costs(prob))
        elif set_model == "links":
            h.set_link_occupancy(True)
        else:
            h.set_copy_engine(4)
        assert dev.evaluate(h, stride, 1 << 18)[-2:] == TWO_PASSES
        groups.add(dev.shapes[-1][0] // 256)
        for n in (1, 255, 256, 257, 512, 513, 1000, 1024):
            assert dev.evaluate(h, stride, n) == TWO_PASSES, (prob.name, set_model, n)
            wavefronts = -(-n // -(-n // 256)) if prob.n_devices <= 6 and prob.n_stages > 3 * prob.n_devices else n
            waves = -(-wavefronts // 256)
            assert dev.shapes[-1] == (-(-wavefronts // waves), 64 * waves), (prob.name, set_model, n)
        assert dev.evaluate(h, stride, 1025) == TWO_PASSES
        assert dev.waves[-1] < 1025 / 2
        h.close()
    assert groups >= {1, 2}


def test_small_batches_of_variants(stub):
    chains = [chain_problem(D, m, v=v, f=3, b=5, w=2, comm=2) for D, m, v in ((7, 20, 3), (11, 45, 3), (3, 6, 1), (6, 20, 3), (2, 30, 4), (6, 12, 4), (7, 12, 4))]
    copy = chain_problem(3, 40, v=1, f=3, b=4, w=2, comm=1)
    copy.dur[O], copy.dur[L] = 2, 3
    run(stub, "small_batches_of_variants", [(prob, model) for prob in chains for model in ("costs", "links")] + [(copy, "copy")])


def where_rows_stand(dev, problems):
    # of a workgroup with one wavefront and one with more, what both have is the rows and, under links, a word for each of the image's
    with_columns = set()
    for prob in problems:
        D, v = prob.n_devices, max(np.bincount(prob.stage_device))
        h = fp.Problem(prob, 512, device=0)
        h.set_link_occupancy(True)
        lds, waves = [], []
        for n in (1, 1 << 20):
            assert dev.evaluate(h, 512, n)[-2:] == TWO_PASSES
            lds.append(dev.lds[-1])
            waves.append(dev.shapes[-1][1] // 64)
        h.close()
        assert waves[0] == 1 < waves[1]
        rows = lds[0] - (lds[1] - lds[0]) // (waves[1] - 1) - 32 * D * 4
        if rows != 32 * D * 16:   # (not as in the image: sixteen columns, of both halves in one from three stages on)
            assert D > 2 and 16 % ((D + 1) // 2) == 0 and rows == 32 * 16 * 16 * (1 if v <= 2 else 2), (prob.name, rows)
            with_columns.add((D, v <= 2))
    # (16 devices of one or two stages take as much either way)
    assert with_columns >= {(4, True), (8, True), (8, False), (16, False), (32, True)}, with_columns


def test_where_the_rows_of_the_timing_pass_stand(stub):
    run(stub, "where_rows_stand", [chain_problem(D, m, v=v, f=3, b=5, w=2, comm=2)
                                   for D in (1, 2, 3, 4, 5, 7, 8, 12, 15, 16, 32, 33, 40) for v in (1, 2, 3, 4) for m in (5, 20, 30)])


ALONE = 6   # (of the timing pass's template arguments: 1 + the bits of the chunk field that select a chunk's states, both passes in one launch)


def both_passes_in_one_launch(dev, cases):
    CU = 256
    for prob, stride, per_cu in cases:
        D, bits = prob.n_devices, {1: 0, 2: 1, 3: 2, 4: 2}[max(np.bincount(prob.stage_device))]
        h = fp.Problem(prob, stride, device=0)
        room = min(64 // D, h.info()["candidates_per_wave"])
        most = room * CU * per_cu
        for n in (1, 63, most + 1, 2 * most):
            assert dev.evaluate(h, stride, n)[-2:] == TWO_PASSES and dev.forms[-1][ALONE] == 0, (prob.name, n)
        for n in (64, 65, CU, CU + 1, 4 * CU, 4 * CU + 1, 16 * CU, 16 * CU + 1, most // 2 + 1, most):
            if n > most:
                continue
            assert dev.evaluate(h, stride, n) == ["time_lists_kernel"] and dev.forms[-1][ALONE] == 1 + bits, (prob.name, n)
            # a SIMD's share of the candidates to a wavefront, or a compute unit's; one workgroup to a compute unit
            share = -(-n // CU) if bits == 2 and prob.n_stages == 4 * D and D <= 6 and n <= 16 * CU else -(-n // (4 * CU))
            wavefronts = -(-n // min(share, room))
            waves = -(-wavefronts // CU)
            assert dev.shapes[-1] == (-(-wavefronts // waves), 64 * waves), (prob.name, n, dev.shapes[-1])
            assert dev.lds[-1] <= 160 * 1024
        h.close()


def test_both_passes_in_one_launch(stub):
    def chain(D, m, v):
        return chain_problem(D, m, v=v, f=3, b=5, w=2, comm=2)
    # with columns, or one or two devices, rows of more than 128 words and no more; without
    run(stub, "both_passes_in_one_launch", [(chain(8, 32, 2), 200, 4), (chain(8, 32, 2), 128, 8), (chain(1, 40, 2), 256, 4), (chain(2, 20, 1), 64, 8),
                                            (chain(16, 64, 2), 392, 4), (chain(12, 40, 2), 256, 8), (chain(24, 30, 2), 192, 8), (chain(5, 8, 4), 136, 8),
                                            (chain(4, 8, 4), 96, 8), (two_tower_problem(m=6), 64, 8)])


def one_launch_does_not_fit(dev, prob, stride):
    h = fp.Problem(prob, stride, device=0)
    assert h.info()["candidates_per_wave"] >= 8 == 64 // prob.n_devices   # (up to 8,192 candidates there would be one launch)
    for n, want in ((256, ["time_lists_kernel"]), (4096, ["time_lists_kernel"]), (8192, TWO_PASSES)):   # (one, four, eight to a wavefront)
        assert dev.evaluate(h, stride, n) == want, n
    h.close()


def test_one_launch_that_does_not_fit(stub):
    run(stub, "one_launch_does_not_fit", chain_problem(8, 150, v=4, f=3, b=5, w=2, comm=2), 1808)


def models_that_keep_two_launches(dev, prob, costs):
    wide = chain_problem(6, 8, v=2, f=3, b=5, w=2, comm=2)
    wide.dur[:] = wide.dur * 100_000
    h = fp.Problem(wide, 64, device=0)
    assert dev.evaluate(h, 64, 500) == ["time_lists_kernel"] and dev.forms[-1][1] == 1
    h.close()
    h = fp.Problem(prob, 64, device=0)
    assert dev.evaluate(h, 64, 500) == ["time_lists_kernel"]
    h.set_link_occupancy(True)
    assert dev.evaluate(h, 64, 500) == TWO_PASSES
    h.set_microbatch_costs(costs)
    assert dev.evaluate(h, 64, 500) == TWO_PASSES
    h.set_link_occupancy(False)
    assert dev.evaluate(h, 64, 500) == TWO_PASSES
    h.close()


def test_models_that_keep_two_launches(stub):
    prob = chain_problem(6, 8, v=2, f=3, b=5, w=2, comm=2)
    run(stub, "models_that_keep_two_launches", prob, workloads.microbatch_costs(prob))


def sliding_generator(dev, full, problems, orders):
    N_CLASSES = 6   # (its place among the generator's arguments)
    dev.stub.stub_watch(b"generate_kernel", N_CLASSES)

    def launched(prob, n):
        h = fp.Problem(prob, 256, device=0)
        dev.launched(dev.lib.fpsched_generate_slide_evaluate(h._h, 4096, 4096, n, dev.results, 4096, 4096, 4096, 1 << 20, None))
        h.close()
        return dev.waves[-1]
    for prob in problems:
        # as many sets to a wavefront as there are lanes for; up to a set for each SIMD, one
        assert launched(prob, full) == -(-full // (64 // prob.n_devices)), prob.name
        degree = max(np.bincount(prob.edge_src).max(), np.bincount(prob.edge_dst).max())
        assert dev.forms[-1][2] == 2 and (dev.forms[-1][1] == 2) == (degree == 2), prob.name
        assert launched(prob, 1024) == 1024, prob.name
    os.environ["FPSCHED_GEN_WAVES"] = "1"
    for prob, n, per_wave, classes in orders:
        assert launched(prob, n) == min(256, -(-n // per_wave)), (prob.name, n)
        assert dev.words[-1] == classes, (prob.name, n, dev.words[-1])


def test_sliding_generator(stub):
    import test_gpu_generate_slide_shared as t
    run(stub, "sliding_generator", t.FULL, [prob for _, prob in t.graphs()] + [prob for _, prob in t.deep_stashes()],
        [(t.placed_chain(D, v, m, 1, seed=D), n, per_wave, classes) for D, v, m, n, per_wave, classes in t.ORDERS])


def segments(dev, rows, device_by_device, spread):
    for prob, stride, beyond in rows:
        h = fp.Problem(prob, stride, device=0)
        room = h.info()["candidates_per_wave"]
        n = beyond(prob.n_devices, room)
        assert dev.evaluate(h, stride, n)[-2:] == TWO_PASSES and room >= min(64 // -(-prob.n_devices // 2), 16)   # (lanes are of two devices)
        blocks, threads = dev.shapes[-1]
        assert (blocks - 1) * threads // 64 * room < n, (prob.name, dev.shapes[-1], room)
        for set_model in (lambda: h.set_link_occupancy(True), lambda: h.set_microbatch_costs(workloads.microbatch_costs(prob)), lambda: h.set_link_occupancy(False)):
            set_model()
            assert dev.evaluate(h, stride, spread + 300) == TWO_PASSES
            assert dev.waves[-1] <= (spread + 300) / min(64 // -(-prob.n_devices // 2), 16) + 256, (prob.name, dev.waves[-1])
        h.close()
    for prob, stride in device_by_device:
        h = fp.Problem(prob, stride, device=0)
        for n in (64, 300, spread):
            assert dev.evaluate(h, stride, n) == ["time_lists_kernel"], (prob.name, n)
        # in two launches: the LDS of the order pass is a wavefront's states, and the rows and two words more of each device, no columns
        D, m = prob.n_devices, prob.n_microbatches
        assert dev.evaluate(h, stride, 1 << 20)[-2:] == TWO_PASSES
        waves = dev.shapes[-2][1] // 64
        states = 64 * 4 * (-(-(m + 1) * (2 if prob.n_stages <= 2 * D else 4) // 4) | 1)
        assert dev.lds[-2] - waves * states == -(-(2 * 32 * D + 2 * D) * 4 // 16) * 16, prob.name
        h.close()


def test_several_candidates_to_a_wavefront(stub):
    import test_gpu_list_segments as t
    chains = [(chain_problem(D, m, v=v, f=3, b=5, w=2, comm=2), -(-3 * v * m // 8) * 8 + 8, t.beyond_one_launch) for D, v, m in t.ROWS]
    run(stub, "segments", chains, [(chain_problem(D, m, v=v, f=3, b=5, w=2, comm=2), -(-3 * v * m // 8) * 8 + 8) for D, v, m in t.DEVICE_BY_DEVICE], t.SPREAD)
