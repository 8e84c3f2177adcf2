"""fpsched_evaluate on a problem with times beyond 24 bits takes calls without a workspace, as the general kernel does."""
import numpy as np
import pytest

import oracle
import workloads
from gpu_common import assert_same
from test_gpu_lists import spec_of
from workloads.problem import chain_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scale", [1, 1000])
@pytest.mark.parametrize("kernel", ["auto", "slots", "general"])
def test_calls_without_a_workspace(kernel, scale):
    import torch
    import paper_2510_05112_amd as fp
    prob = chain_problem(8, 32, v=2, f=30 * scale, b=50 * scale, w=20 * scale, comm=45, mem_cap=12)
    words = workloads.generate(spec_of(prob, 64, 3), threads=4)
    h = fp.Problem(prob, words.shape[2], device=0)
    h.select_kernel(kernel)
    ops, res = torch.from_numpy(words.view(np.int16)).cuda(), h.alloc_results(len(words))
    lib, stream = fp.load_library(), h._stream(None)
    ref = oracle.evaluate(prob, words)
    for pointer, size in ((0, 0), (ops.data_ptr() + 2, 4096), (ops.data_ptr(), 8)):   # none, misaligned, too small
        rc = lib.fpsched_evaluate(h._h, ops.data_ptr(), len(words), words.shape[2], h._res_struct(res), pointer, size, stream)
        if scale == 1 and kernel != "general":
            assert rc == (-2 if size == 8 else -1)
        else:
            assert rc == 0
            torch.cuda.synchronize()
            assert_same({name: t.cpu().numpy() for name, t in res.items()}, ref, f"{kernel} x {scale}")
            for t in res.values():
                t.zero_()
    h.evaluate(ops, res)
    assert_same({name: t.cpu().numpy() for name, t in res.items()}, ref, f"{kernel} x {scale}, with a workspace")
    h.close()
