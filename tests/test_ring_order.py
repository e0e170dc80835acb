"""The kernels that stream through rings of LDS stages wait with counted s_waitcnt vmcnt(n):
the n youngest loads may still be in flight.  That is right only if the stages' loads are
sent in ring order, and the scheduler may interleave the first ones, which go to
distinct LDS objects, unless a scheduling barrier stands between them.  CPU only."""
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2606_21712_amd", "csrc")
# a ring's first loads: issue(st0, 0); issue(st1, 1); ... (the later ones are sent inside a step)
FIRST = re.compile(r"(?:if constexpr \(S == 4\) )?\bissue\(st(\d), (\d)[^;]*\);")


def code(name):
    with open(os.path.join(CSRC, name)) as f:
        return re.sub(r"//[^\n]*", "", f.read())


def ring_sources():
    return sorted(n for n in os.listdir(CSRC) if n.endswith(".hip") and "wait_vm(" in code(n))


def test_ring_sources_found():
    assert {"ffn_stream.hip", "ffn_f32.hip", "router.hip"} <= set(ring_sources())


@pytest.mark.parametrize("name", ring_sources())
def test_first_loads_are_pinned(name):
    text = code(name)
    found = [m for m in FIRST.finditer(text) if m.group(1) == m.group(2)]
    later = [(a, b) for a, b in zip(found, found[1:]) if int(b.group(2)) == int(a.group(2)) + 1]
    assert later, "no ring prologue found"
    for a, b in later:
        between = text[a.end():b.start()]
        assert "__builtin_amdgcn_sched_barrier(0);" in between, text[a.start():b.end()]
