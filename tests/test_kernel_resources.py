"""What the compiler gives the kernels of the main path: nothing of a lane's lives in memory.  (A form at the limit of its vector
registers takes to it silently, and its loop waits for loads that no source line shows.)"""
import re

import pytest

from test_inline_asm import SOURCES, compiled, pytestmark  # noqa: F401


@pytest.mark.parametrize("name", SOURCES)
def test_no_scratch_memory(name):
    text = compiled(name)
    metadata = text[text.index("amdhsa.kernels:"):]
    kernels = re.findall(r"\.name: +(\S+)\n\s+\.private_segment_fixed_size: (\d+)", metadata)
    assert len(kernels) == metadata.count(".vgpr_spill_count:") > 0
    assert [k for k in kernels if k[1] != "0"] == []
    assert set(re.findall(r"\.vgpr_spill_count: +(\d+)", metadata)) == {"0"}
