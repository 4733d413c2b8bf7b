"""A shared-memory array that a kernel reads or writes as a wider vector than
its element is declared with that alignment: the compiler may emit one access
of the vector's size, and the layout of LDS promises an array no more than what
its declaration asks for."""
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2104_12922_amd", "csrc")
SIZE = {"float": 4, "int": 4, "uint32_t": 4, "uint16_t": 2, "double": 8, "float2": 8, "uint2": 8,
        "double2": 16, "float4": 16, "uint4": 16, "bf16x8": 16}
SOURCES = sorted(f for f in os.listdir(CSRC) if f.endswith((".hip", ".h", ".cpp")))


def shared_arrays(txt):
    """(element bytes, declared alignment, name) of every __shared__ array."""
    for decl in re.findall(r"__shared__\s+([^;]+);", txt):
        m = re.match(r"(?:__align__\((\d+)\)\s*|alignas\((\d+)\)\s*)?(\w+)\s+(.*)", decl, re.S)
        if not m or "<" in decl:          # a structure of its own (its members say their alignment)
            continue
        align = int(m.group(1) or m.group(2) or 0)
        for name in re.findall(r"(\w+)\s*\[", m.group(4)):
            yield SIZE.get(m.group(3)), align, name


@pytest.mark.parametrize("source", SOURCES)
def test_vector_accesses_are_declared(source):
    txt = re.sub(r"//[^\n]*", "", open(os.path.join(CSRC, source)).read())
    for element, align, name in shared_arrays(txt):
        for vec in re.findall(r"reinterpret_cast<(?:const )?(\w+)\s*\*>\(&?%s\b" % name, txt):
            if element and vec in SIZE:
                assert max(element, align) >= SIZE[vec], f"{source}: {name} accessed as {vec}"
