"""Rules that the device code keeps, read off its source on the CPU."""
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2605_08134_amd", "csrc")
SOURCES = sorted(f for f in os.listdir(CSRC) if f.endswith((".hip", ".h")))


def _code(name):
    text = open(os.path.join(CSRC, name)).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return re.sub(r"//[^\n]*", "", text)


@pytest.mark.parametrize("name", SOURCES)
def test_no_workgroup_waits_for_another(name):
    """Workgroups that share work hand it over to the last one to arrive: no loop polls memory, so
    whatever a counter holds, every launch ends."""
    assert not re.search(r"(while|for)\s*\([^{};]*__hip_atomic_load", _code(name))
    assert "s_sleep" not in _code(name)


@pytest.mark.parametrize("name", SOURCES)
def test_arrival_counters_wrap_by_themselves(name):
    """The arrival that is last takes the counter back to 0 in the same operation: a store of 0 beside
    it could fall between the arrivals of two overlapping calls and leave the counter off for good."""
    assert "__hip_atomic_store" not in _code(name)


@pytest.mark.parametrize("name", SOURCES)
def test_inline_assembly_leaves_m0_to_the_compiler(name):
    """Loads into LDS take their address from M0, and so do things of the compiler's own: an asm
    statement gets it as an operand and writes it behind nobody's back."""
    for stmt in re.findall(r"asm\s+volatile\s*\((.*?)\)\s*;", _code(name), flags=re.S):
        assert not re.search(r"\bm0\s*,", stmt), stmt
        if "load_lds" in stmt:
            assert '"{m0}"' in stmt, stmt


def test_ping_pong_groups_part_after_their_first_reads():
    """gemm_tile_pp: group 1 falls one barrier behind once its first fragment reads have returned; the
    region they come from may be refilled from that barrier on."""
    code = _code("gemm_bf16.hip")
    start = code.index("read_b(0, 0, 0);")
    assert re.match(r'read_b\(0, 0, 0\);\s*if \(grp == 1\) asm volatile\("s_waitcnt lgkmcnt\(0\)\\n\\ts_barrier"',
                    code[start:])
