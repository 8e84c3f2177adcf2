"""``tuner.tune`` goes through lists where the kernels that time schedules while they generate them do not take the
problem or the cost model, and only there."""
import gc

import pytest

from paper_2510_05112_amd import tuner
from test_tuner import chain

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def problem():
    return chain(4, 2, 10, "circular")


@pytest.fixture(autouse=True)
def collect():
    """The caught errors' frames hold device tensors in reference cycles: gone before another test counts allocations."""
    yield
    gc.collect()


class Refusing:
    """A handle one of whose generate_evaluate calls fails with `code`; counts what is generated as lists."""

    def __init__(self, handle, code, failing_call):
        self.handle, self.code, self.failing_call = handle, code, failing_call
        self.calls = self.lists = 0

    def __getattr__(self, name):
        return getattr(self.handle, name)

    def generate_evaluate(self, *args, **kwargs):
        from paper_2510_05112_amd import FpschedError
        self.calls += 1
        if self.calls == self.failing_call:
            raise FpschedError(self.code, "fpsched_generate_evaluate")
        return self.handle.generate_evaluate(*args, **kwargs)

    def generate(self, *args, **kwargs):
        self.lists += 1
        return self.handle.generate(*args, **kwargs)


@pytest.mark.parametrize("failing_call", [1, 2])
@pytest.mark.parametrize("code", [-6, -4, -3, -2, -1])
def test_which_errors_lead_to_the_list_path(problem, code, failing_call):
    import paper_2510_05112_amd as fp
    h = fp.Problem(problem, tuner.stride_for(problem), device=0)
    refusing = Refusing(h, code, failing_call)
    if code in (-6, -4):   # unsupported, time bound
        assert tuner.tune(refusing, problem, True, slide=True) == tuner.tune(h, problem, True, slide=True)
        assert refusing.lists == 1
    else:                  # a HIP error, no memory, a bad argument
        with pytest.raises(fp.FpschedError) as e:
            tuner.tune(refusing, problem, True, slide=True)
        assert e.value.code == code and refusing.lists == 0
    h.close()


def test_a_stride_the_handle_was_not_made_for_is_refused(problem):
    import paper_2510_05112_amd as fp
    h = fp.Problem(problem, tuner.stride_for(problem) - 8, device=0)
    with pytest.raises(fp.FpschedError) as e:
        tuner.tune(h, problem, True)
    assert e.value.code == -1 and "fpsched_evaluate" in str(e.value)
    h.close()
