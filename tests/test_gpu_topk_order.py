"""Top-k: the time does not depend on the order of the values, nor does it grow with the batch as one workgroup's chain of
sorts; results at the sizes where a batch gets one part, one launch, or one sort more."""
import numpy as np
import pytest

from test_gpu_select import handle, values  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


def results_of(ms, flags):
    import torch
    return dict(makespan=torch.from_numpy(ms).cuda(), idle=torch.zeros(1, dtype=torch.int64).cuda(),
                peak=torch.zeros(1, dtype=torch.int32).cuda(), flags=torch.from_numpy(flags).cuda())


def best_time(handle, ms, k):
    """Least time of a few calls, in us."""
    import torch
    res = results_of(ms, np.zeros(len(ms), np.uint8))
    ws = handle.alloc_workspace(len(ms), k)
    out = handle.topk(res, k, ws)
    times = []
    for _ in range(8):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        handle.topk(res, k, ws, out)
        b.record()
        torch.cuda.synchronize()
        times.append(1000 * a.elapsed_time(b))
    return min(times)


def test_falling_values_take_about_as_long_as_random_ones(handle):  # noqa: F811
    # (measured: 1.1 times as long; 6 times when a part was walked from front to back)
    n, rng = 1 << 20, np.random.default_rng(1)
    order = np.arange(n, dtype=np.int64)
    assert best_time(handle, order[::-1].copy(), 128) < 3 * best_time(handle, rng.permutation(order), 128)


def test_large_batches_get_more_parts_not_longer_ones(handle):  # noqa: F811
    # (measured: 2 times as long for 64 times the values; 34 times with at most 64 parts and a sort per batch of elements)
    rng = np.random.default_rng(2)
    small, large = (best_time(handle, rng.permutation(np.arange(n, dtype=np.int64)), 1024) for n in (1 << 16, 1 << 22))
    assert large < 8 * small


# one workgroup's limit of 16 sorts' worth of elements: 16 x 1024 up to k = 512, 16 x 2048 at k = 1024, for a part and for
# what the parts leave; 8 to 64 parts below that
@pytest.mark.parametrize("kind", ["random", "falling", "ties", "wide"])
@pytest.mark.parametrize("n,k", [(8 * 16384, 300), (8 * 16384 + 1, 300), (64 * 16384 + 1, 7), (8 * 32768, 1024), (8 * 32768 + 1, 1024),
                                 (32 * 32768, 1024), (32 * 32768 + 1, 1024), (128 * 16384 + 1, 128), (33 * 16384 - 5, 512)])
def test_results_at_the_edges(handle, n, k, kind):  # noqa: F811
    rng = np.random.default_rng(n)
    ms = values(kind, n, rng)
    flags = np.where(rng.random(n) < 0.9, 0, rng.integers(1, 8, n)).astype(np.uint8)
    out = {key: t.cpu().numpy() for key, t in handle.topk(results_of(ms, flags), k).items()}
    ok = np.flatnonzero(flags == 0)
    best = ok[np.argsort(ms[ok], kind="stable")[:k]]
    assert out["count"][0] == k
    np.testing.assert_array_equal(out["idx"], best)
    np.testing.assert_array_equal(out["makespan"], ms[best])
