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
