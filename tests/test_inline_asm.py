"""What the compiler cannot see of the kernels' inline assembly, read from what it makes of them: a statement that reads LDS
waits for it before it ends (the registers would else be used, or copied, while the value is still on its way), and an output
that is written while inputs are still to be read has no register with one of them in common."""
import os
import re
import subprocess

import pytest

from paper_2510_05112_amd import build

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
SOURCES = [name for name in build.SOURCES if r"\n\t" in open(os.path.join(build.CSRC, name)).read()]
pytestmark = pytest.mark.skipif(not os.path.exists(HIPCC), reason="no hipcc")


def compiled(name, *what):
    flags = [f for f in build.FLAGS if f not in ("-fPIC", "-shared")]
    cmd = [HIPCC] + flags + ["--cuda-device-only", "-S", *what, "-o", "-", os.path.join(build.CSRC, name)]
    return subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.DEVNULL, text=True, check=True).stdout


@pytest.mark.parametrize("name", SOURCES)
def test_no_lds_read_is_in_flight_at_the_end_of_a_statement(name):
    n_reads, unwaited = 0, []
    for statement in re.findall(r";;#ASMSTART\n(.*?);;#ASMEND", compiled(name), re.S):
        waits = True
        for line in statement.split("\n"):
            if line.strip().startswith("ds_read"):
                n_reads, waits = n_reads + 1, False
            elif "s_waitcnt" in line and "lgkmcnt(0)" in line:
                waits = True
        if not waits:
            unwaited.append(statement)
    assert not unwaited, f"{len(unwaited)} statements, the first:\n{unwaited[0]}"
    assert n_reads > 100 or name != "timing.hip"


@pytest.mark.parametrize("name", SOURCES)
def test_outputs_of_several_instructions_share_no_register_with_an_input(name):
    statements = set(re.findall(r'asm sideeffect "((?:[^"\\]|\\.)*)", "([^"]*)"', compiled(name, "-emit-llvm")))
    several = [(text, constraints) for text, constraints in statements if r"\0A" in text]
    assert several
    for text, constraints in several:
        shared = [c for c in constraints.split(",") if c.startswith("=") and "&" not in c]
        assert not shared, (shared, text[:200].replace(r"\0A\09", "; "))
