"""fpsched_problem_info describes one kernel: what it says of lanes and candidates fits a wavefront."""
import pytest

from workloads.problem import chain_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kernel", ["slots", "general"])
@pytest.mark.parametrize("D", [1, 2, 3, 16, 17, 32, 33, 64])
def test_lanes_and_candidates_fit_a_wavefront(D, kernel):
    import paper_2510_05112_amd as fp
    h = fp.Problem(chain_problem(D, 8), 24, device=0)
    h.select_kernel(kernel)
    info = h.info()
    assert info["lanes_per_candidate"] >= (D + 1) // 2 and info["candidates_per_wave"] >= 1
    assert info["lanes_per_candidate"] * info["candidates_per_wave"] <= 64
    h.close()
