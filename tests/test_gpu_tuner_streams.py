"""The tuner's two generator forms side by side on two streams: no memory of the one is the other's, and a grid of many more sets
than segments (whose counters and class marks are looked at all the time) ranks as the two forms one after the other do."""
import numpy as np
import pytest

from test_gpu_topk_order import results_of
from workloads.problem import chain_problem

pytestmark = pytest.mark.gpu


def test_memory_of_the_two_forms(monkeypatch):
    import paper_2510_05112_amd as fp
    from paper_2510_05112_amd import tuner
    prob = chain_problem(4, 8, f=2, b=3, w=2, comm=1)
    handle = fp.Problem(prob, tuner.stride_for(prob), device=0)
    call, used = fp.Problem.generate_evaluate, []

    def noted(self, policy, inflight, results=None, out=None, workspace=None, stream=None, slide=False):
        if workspace is None:
            workspace = self.alloc_workspace(len(policy), 0)
        got = call(self, policy, inflight, results, out, workspace, stream, slide)
        # (numbers: a tensor kept here would keep its memory)
        used.append([(t.data_ptr(), t.data_ptr() + t.numel() * t.element_size()) for t in (workspace, *got[0].values(), *got[1].values())])
        return got
    monkeypatch.setattr(fp.Problem, "generate_evaluate", noted)
    rng = np.random.default_rng(5)
    limits = rng.integers(1, 9, (8000, prob.n_stages)).astype(np.int32)
    best = tuner.tune(handle, prob, False, k=64, inflight_options=list(limits), slide=True)
    assert len(used) == 2
    for lo, hi in used[0]:
        for a, b in used[1]:
            assert hi <= a or b <= lo
    monkeypatch.undo()
    # one after the other
    import torch
    _, pol, inf = tuner.grid(prob, False, list(limits), False)
    d_pol, d_inf = torch.from_numpy(pol).cuda(), torch.from_numpy(inf).cuda()
    both = [handle.generate_evaluate(d_pol, d_inf, slide=slide)[0] for slide in (False, True)]
    ms, flags = (torch.cat([r[name] for r in both]).cpu().numpy() for name in ("makespan", "flags"))
    top = handle.topk(results_of(ms, flags), 64)
    count = int(top["count"].item())
    assert len(best) == count and count > 0
    n = len(pol)
    assert [(b["makespan"], b["index"] + n * b["slid"]) for b in best] == \
        list(zip(top["makespan"].tolist()[:count], top["idx"].tolist()[:count]))
