"""Top-k and Pareto front over values a caller supplies: sizes around one part, one sort and one tile, orders in which
every candidate or none displaces the ones before it, values that do and do not fit in 32 bits, ties, no candidates."""
import numpy as np
import pytest

import oracle
from workloads.problem import chain_problem

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def handle():
    import paper_2510_05112_amd as fp
    return fp.Problem(chain_problem(2, 4), 16, device=0)


def values(kind, n, rng):
    return {"random": rng.integers(0, 1 << 31, n), "ties": rng.integers(0, 3, n), "rising": np.arange(n),
            "falling": np.arange(n)[::-1], "wide": rng.integers(0, 5, n) << 32, "negative": rng.integers(-5, 5, n),
            "edge": 0xfffffffe + rng.integers(0, 2, n)}[kind].astype(np.int64)


@pytest.mark.parametrize("kind", ["random", "ties", "rising", "falling", "wide", "negative", "edge"])
@pytest.mark.parametrize("n", [1, 63, 128, 129, 1023, 2048, 2049, 4097, 20011, 150001])
def test_topk(handle, kind, n):
    import torch
    rng = np.random.default_rng(n)
    ms = values(kind, n, rng)
    for k, feasible in ((1, 0.9), (5, 0.002), (64, 1.0), (65, 0.5), (512, 0.9), (1024, 0.7), (300, 0.0)):
        flags = np.where(rng.random(n) < feasible, 0, rng.integers(1, 8, n)).astype(np.uint8)
        res = dict(makespan=torch.from_numpy(ms).cuda(), idle=torch.zeros(1, dtype=torch.int64).cuda(),
                   peak=torch.zeros(1, dtype=torch.int32).cuda(), flags=torch.from_numpy(flags).cuda())
        out = {key: t.cpu().numpy() for key, t in handle.topk(res, k).items()}
        ok = np.flatnonzero(flags == 0)
        best = ok[np.lexsort((ok, ms[ok]))][:k]
        assert out["count"][0] == len(best), (k, feasible)
        np.testing.assert_array_equal(out["idx"], np.concatenate([best, np.full(k - len(best), -1)]))
        np.testing.assert_array_equal(out["makespan"], np.concatenate([ms[best], np.full(k - len(best), np.iinfo(np.int64).max)]))


@pytest.mark.parametrize("n,points", [(1, 1), (2048, 2048), (2049, 2049), (6000, 2048), (6000, 2049), (50000, 300), (50000, 5000)])
@pytest.mark.parametrize("scale", [1, 1 << 33])
def test_pareto(handle, n, points, scale):
    """`points` candidates on one falling front, in a random order among dominated ones: tile fronts that fit in one
    tile together, or do not."""
    import torch
    rng = np.random.default_rng(n + points)
    t = rng.integers(0, points, n)
    t[rng.permutation(n)[:points]] = np.arange(points)
    late = rng.integers(0, 2, n) * (rng.random(n) < 0.5)
    res = dict(makespan=((t + late) * scale).astype(np.int64), idle=np.zeros((n, 2), np.int64),
               peak=np.stack([points - t, rng.integers(0, 2, n)], 1).astype(np.int32),
               flags=rng.choice([0, 0, 0, 2, 4], n).astype(np.uint8))
    for kmax in (1, 64, 1024):
        out = {key: x.cpu().numpy() for key, x in handle.pareto({key: torch.from_numpy(x).cuda() for key, x in res.items()}, kmax).items()}
        idx, ms, pk, cnt = oracle.pareto(res, kmax)
        assert out["count"][0] == cnt
        for got, want in ((out["idx"], idx), (out["makespan"], ms), (out["peak"], pk)):
            np.testing.assert_array_equal(got[:cnt], want[:cnt])
        assert (out["idx"][cnt:] == -1).all()
