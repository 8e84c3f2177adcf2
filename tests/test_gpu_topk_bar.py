"""Top-k: the bar that a part's first batches give, where the k smallest sit in one wavefront, in one lane, or nearly alone, and
at the sizes from which on it is used."""
import numpy as np
import pytest

from test_gpu_select import handle  # noqa: F401  (fixture)
from test_gpu_topk_order import results_of

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("where", ["wavefront", "lane", "few", "same", "wide"])
@pytest.mark.parametrize("k", [1, 31, 32, 33, 64, 100, 512])
def test_bar(handle, k, where):  # noqa: F811
    rng = np.random.default_rng(k)
    for n in (128, 129, 4 * k - 1, 4 * k, 4 * k + 1, 2048, 2049, 40000):
        at = np.arange(n)
        ms = rng.integers(1000, 100000, n)
        flags = np.zeros(n, np.uint8)
        if where == "wavefront":
            ms[at // 64 % 8 == 5] -= 1000
        elif where == "lane":
            ms[at % 64 == 17] -= 1000
        elif where == "few":
            flags[rng.random(n) < 0.97] = 4
        elif where == "same":
            ms[:] = 7
        else:
            ms = ms << 33
        out = {key: t.cpu().numpy() for key, t in handle.topk(results_of(ms.astype(np.int64), flags), k).items()}
        ok = np.flatnonzero(flags == 0)
        best = ok[np.lexsort((ok, ms[ok]))][:k]
        assert out["count"][0] == len(best)
        np.testing.assert_array_equal(out["idx"][:len(best)], best)
        np.testing.assert_array_equal(out["makespan"][:len(best)], ms[best])
        assert (out["idx"][len(best):] == -1).all()
