"""What becomes of the kernels of the main path: nothing of a lane's lives in memory (a form at the limit of its vector registers
takes to it silently, and its loop waits for loads that no source line shows), and the steps begin where they are fastest."""
import os
import re
import subprocess

import pytest

from test_inline_asm import HIPCC, SOURCES, compiled, pytestmark  # noqa: F401


@pytest.mark.parametrize("name", SOURCES)
def test_no_scratch_memory(name):
    text = compiled(name)
    metadata = text[text.index("amdhsa.kernels:"):]
    kernels = re.findall(r"\.name: +(\S+)\n\s+\.private_segment_fixed_size: (\d+)", metadata)
    assert len(kernels) == metadata.count(".vgpr_spill_count:") > 0
    assert [k for k in kernels if k[1] != "0"] == []
    assert set(re.findall(r"\.vgpr_spill_count: +(\d+)", metadata)) == {"0"}


def test_place_of_the_rounds_in_memory(tmp_path):
    """The statement of the rounds begins at a multiple of 32 bytes, with synchronisation 16 behind one, whatever the code in front of it."""
    source, made = str(tmp_path / "timing.s"), str(tmp_path / "timing.o")
    with open(source, "w") as f:
        f.write(compiled("timing.hip").replace(".Lrounds_", "rounds_"))   # (a symbol that the assembler keeps)
    llvm = os.path.join(os.path.dirname(os.path.realpath(HIPCC)), "..", "llvm", "bin")
    subprocess.run([os.path.join(llvm, "clang"), "-target", "amdgcn-amd-amdhsa", "-mcpu=gfx950", "-c", "-o", made, source], check=True)
    symbols = subprocess.run([os.path.join(llvm, "llvm-readelf"), "-sW", made], stdout=subprocess.PIPE, text=True, check=True).stdout
    places = {int(form): int(at, 16) % 32 for at, form in re.findall(r"^ +\d+: ([0-9a-f]+) .* rounds_(\d+)$", symbols, re.M)}
    sync = 33   # (second edges and synchronisation)
    assert len(places) == 10 and places.pop(sync) == 16 and set(places.values()) == {0}
