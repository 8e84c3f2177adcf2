"""Pareto front: what a tile drops before it sorts, at the edges of the classes that it sorts peaks into."""
import numpy as np
import pytest

import oracle
from test_pareto import check_front, synthetic_results
from workloads.problem import chain_problem


@pytest.mark.gpu
@pytest.mark.parametrize("peaks", [(0, 2), (0, 70), (60, 68), (1000, 1200), (1 << 20, 1 << 24), ((1 << 31) - 300, (1 << 31) - 1)])
@pytest.mark.parametrize("makespans", [(0, 3), (100, 160), (1, 1 << 40), (oracle.INT64_MAX - 2, oracle.INT64_MAX)])
def test_front_of_ties_and_close_peaks(peaks, makespans):
    """Classes of one peak and of many, the largest peaks, equal pairs in one tile and in several, the largest times."""
    import torch

    import paper_2510_05112_amd as fp
    handle = fp.Problem(chain_problem(2, 4), 16, device=0)
    for n in (1, 2, 63, 1025, 2048, 2049, 70001):
        res = synthetic_results(n, 2, n, makespans, peaks)
        res["makespan"][(res["flags"] & 3 == 0) & (np.arange(n) % 7 == 0)] = makespans[1]
        out = {key: x.cpu().numpy() for key, x in handle.pareto({key: torch.from_numpy(x).cuda() for key, x in res.items()}, 300).items()}
        check_front(res, 300, out["idx"], out["makespan"], out["peak"], int(out["count"][0]))
