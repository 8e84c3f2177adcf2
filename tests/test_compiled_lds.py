"""What the compiler makes of kernels where lanes hand one another values through LDS, or store in halves and read in dwords."""
import re

import pytest

from test_inline_asm import compiled, pytestmark  # noqa: F401


@pytest.fixture(scope="module")
def generator():
    return compiled("generate.hip", "-emit-llvm")


def kernels(text):
    return re.findall(r"define [^\n]*@\w*generate_kernelILi(\d)ELi(\d)ELi(\d)E[^\n]*\n(.*?)\n}\n", text, re.S)


def test_where_the_stages_are_is_read_behind_a_barrier(generator):
    found = [body for v, graph, _, body in kernels(generator) if (v, graph) == ("2", "3")]
    assert len(found) == 3
    for body in found:
        start = body.split("call void @llvm.amdgcn.s.barrier()")
        assert len(start) == 2
        parts = re.split(r'fence syncscope\("wavefront[^"]*"\) acq_rel[^\n]*\n\s*(?:tail )?call void @llvm\.amdgcn\.wave\.barrier\(\)', start[1])
        assert len(parts) == 2
        accesses = re.findall(r"(load|store) i32\b[^\n]*ptr addrspace\(3\)", parts[0])
        assert len(accesses) >= 2 and set(accesses) == {"store"}   # (one per stage)
        assert re.search(r"load i32, ptr addrspace\(3\)", parts[1])


def types_of_halves(text):
    types = dict(re.findall(r"^(!\d+) = !\{(.*)\}$", text, re.M))
    tags = re.findall(r"(?:load|store) i16\b[^\n]*ptr addrspace\(3\)[^\n]*!tbaa (!\d+)", text)
    return [types[types[tag].split(",")[0]].split(",")[0] for tag in tags]


def test_halves_of_words_are_accessed_as_such(generator):
    # counters and staged op words are stored in dwords and read in halves, or the other way round: of a type the compiler takes to be
    # anything, so that no such access moves past one of the other kind
    found = types_of_halves(generator)
    assert len(found) > 100 and set(found) == {'!"omnipotent char"'}
    # the placement's lanes store a row's words in halves, and read them in dwords
    whole = compiled("wslide.hip", "-emit-llvm")
    types = whole[whole.index("\n!0 = "):]
    kernels_there = re.findall(r"define [^\n]*@\w*wslide_place_kernelILb\dE[^\n]*\n(.*?)\n}\n", whole, re.S)
    assert len(kernels_there) == 2
    for body in kernels_there:
        found = types_of_halves(body + types)
        assert len(found) >= 10 and set(found) == {'!"omnipotent char"'}
