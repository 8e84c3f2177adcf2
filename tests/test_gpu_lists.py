"""The two-pass list evaluation (order pass, timing pass) at the sizes where its splits can go wrong: device counts
around the pairs and segments of a wavefront, rows that end at every position of a group of eight words or fill
their stride, state tables that force fewer rows per wavefront, batches that make the order pass draw blocks."""
import numpy as np
import pytest

import workloads
from gpu_common import check_batch
from workloads.problem import F, chain_problem, pack_word

pytestmark = pytest.mark.gpu


def spec_of(prob, n, seed, per_mille=30, recompute=0):
    v = max(1, int(np.bincount(prob.stage_device).max()))
    longest = v * prob.n_microbatches * (3 if prob.has_w else 2) + (prob.n_microbatches if recompute else 0)
    return workloads.Spec(0, prob, n, -(-longest // 8) * 8, 8, recompute=recompute, max_marks_per_device=prob.n_microbatches,
                          cap_units=max(2, prob.n_devices // 2), seed=seed, deadlock_per_mille=per_mille)


@pytest.mark.parametrize("D,v,m", [(1, 1, 5), (2, 1, 8), (3, 2, 4), (5, 1, 9), (14, 2, 10), (17, 2, 16), (21, 1, 6), (22, 2, 5), (31, 1, 4), (33, 1, 5), (40, 1, 8),
                                   (63, 1, 3), (64, 1, 3)])
def test_device_counts(D, v, m):
    prob = chain_problem(D, m, v=v, f=3, b=5, w=2, comm=2, mem_cap=max(2, D // 2))
    # (many copies: several wavefronts per workgroup, and segments that take further candidates)
    words = np.tile(workloads.generate(spec_of(prob, 150, D), threads=8), (1 + 40000 // (150 * D), 1, 1))
    check_batch(prob, words, 8, f"D={D}", kernels=("slots",))


@pytest.mark.parametrize("stop", list(range(0, 26)))
def test_lists_stop_at_every_position(stop):
    """A list cut off, an op that is not legal, or a malformed word at each position, garbage behind the END word."""
    prob = chain_problem(2, 5, v=1, f=2, b=3, w=1, comm=1)
    base = workloads.generate(spec_of(prob, 4, 11, 0), threads=1)
    rows = []
    for bad in (0x0007, pack_word(F, 0, 0), pack_word(F, 1, 0), pack_word(F, 0, 5), pack_word(F, 0, 2047)):
        for d in range(2):
            w = np.zeros((2, 32), np.uint16)
            w[:, :base.shape[2]] = base[1]
            w[d, stop] = bad
            w[d, min(stop + 1, 31):] |= np.uint16(0)
            rows.append(w.copy())
            if bad < 0x2000:
                w[d, stop + 1:] = pack_word(F, 3, 9)
                rows.append(w)
    check_batch(prob, np.stack(rows), 4, f"stop {stop}")


@pytest.mark.parametrize("m,has_w", [(4, True), (8, True), (12, False), (16, True), (32, True), (40, False)])
def test_rows_that_fill_their_stride(m, has_w):
    prob = chain_problem(3, m, v=1, f=2, b=4, w=1 if has_w else None, comm=1)
    spec = spec_of(prob, 300, m)
    spec.stride = -(-(m * (3 if has_w else 2)) // 8) * 8
    check_batch(prob, workloads.generate(spec, threads=8), 8, f"m={m}")


@pytest.mark.parametrize("v,m", [(2, 700), (4, 600), (1, 2048)])
def test_large_state_tables(v, m):
    prob = chain_problem(2, m, v=v, f=1, b=1, w=1, comm=1)
    check_batch(prob, workloads.generate(spec_of(prob, 6, m), threads=6), 4, f"v={v} m={m}", kernels=("slots",))


def test_order_pass_draws_blocks():
    """More than eight blocks of rows per resident wavefront: the further blocks come from the counter."""
    prob = chain_problem(16, 8, v=2, f=3, b=6, w=3, comm=1, mem_cap=9)
    words = workloads.generate(spec_of(prob, 2048, 5, 20, recompute=1), threads=8)
    words = np.tile(words, (64, 1, 1))
    check_batch(prob, words[:131072 - 3], 16, "many blocks", threads=16, kernels=("slots",))


@pytest.mark.parametrize("D,v,m,scale", [(3, 2, 9, 20000), (14, 1, 12, 9000), (33, 2, 6, 1500)])
def test_times_beyond_24_bits(D, v, m, scale):
    prob = chain_problem(D, m, v=v, f=3 * scale, b=5 * scale + 1, w=2 * scale, comm=scale - 1, mem_cap=max(2, D // 2))
    words = np.tile(workloads.generate(spec_of(prob, 150, D), threads=8), (1 + 20000 // (150 * D), 1, 1))
    gpu, _ = check_batch(prob, words, 8, f"D={D}")
    assert gpu["makespan"].min() > 0


def test_times_beyond_24_bits_on_a_dag():
    """Two towers that merge: second inputs and outputs; latencies beyond 16 bits."""
    spec = workloads.config(5, 500)
    prob = spec.problem
    prob.dur = prob.dur * 3001
    prob.edge_comm = prob.edge_comm * 70001
    check_batch(prob, workloads.generate(spec, threads=8), 16, "towers", threads=8)
