"""The rounds of the launch that does both passes begin where those of the timing pass do: at a multiple of 32 bytes."""
import os
import re
import subprocess

from test_inline_asm import HIPCC, compiled, pytestmark  # noqa: F401


def test_place_of_the_rounds_in_memory(tmp_path):
    source, made = str(tmp_path / "timing.s"), str(tmp_path / "timing.o")
    with open(source, "w") as f:
        f.write(compiled("timing.hip").replace(".Lalone_", "alone_"))   # (a symbol that the assembler keeps)
    llvm = os.path.join(os.path.dirname(os.path.realpath(HIPCC)), "..", "llvm", "bin")
    subprocess.run([os.path.join(llvm, "clang"), "-target", "amdgcn-amd-amdhsa", "-mcpu=gfx950", "-c", "-o", made, source], check=True)
    symbols = subprocess.run([os.path.join(llvm, "llvm-readelf"), "-sW", made], stdout=subprocess.PIPE, text=True, check=True).stdout
    places = [int(at, 16) % 32 for at in re.findall(r"^ +\d+: ([0-9a-f]+) .* alone_\d+$", symbols, re.M)]
    assert places == [0] * 9
