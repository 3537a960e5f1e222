"""The rule that picks the kernel of a bf16 attention (csrc/attn_route.h), evaluated on the CPU.  Blocks
laid out on the device cost a walk over all sequences: many short sequences, where that is
longer than the attention itself, must not get there, and long or few ones must."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROBE = r"""
#include <cstdio>
#include <cstdlib>
#include "attn_route.h"
int main(int, char** a) {
  std::printf("%d", (int)dare::attn_route(atol(a[1]), atol(a[2]), atoi(a[3]), atoi(a[4]), atoi(a[5]), atoi(a[6])));
}
"""
NARROW, WIDE, TALL, LAID_OUT = range(4)


@pytest.fixture(scope="module")
def route(tmp_path_factory):
    d = tmp_path_factory.mktemp("attn_route")
    (d / "probe.cpp").write_text(PROBE)
    subprocess.run(["g++", "-std=c++17", "-I", os.path.join(ROOT, "paper_2605_08134_amd", "csrc"), str(d / "probe.cpp"),
                    "-o", str(d / "probe")], check=True)
    return lambda *args: int(subprocess.run([str(d / "probe")] + [str(int(v)) for v in args], capture_output=True,
                                            text=True, check=True).stdout)


@pytest.mark.parametrize("batch,heads,seq,want", [
    (1, 32, 1024, NARROW), (1, 32, 1920, NARROW), (2, 4, 201, NARROW), (4, 8, 1024, NARROW),   # few pairs
    (4, 32, 256, WIDE), (16, 8, 64, WIDE), (8, 16, 128, WIDE),                       # one round whatever is refreshed
    (3, 32, 777, LAID_OUT), (2, 32, 512, LAID_OUT), (8, 32, 2048, LAID_OUT), (16, 32, 256, LAID_OUT),
    (32, 32, 512, LAID_OUT), (64, 8, 1024, LAID_OUT),
    (32, 32, 128, WIDE), (64, 32, 64, WIDE), (64, 4, 256, WIDE), (128, 32, 64, WIDE), (256, 32, 64, WIDE),
    (512, 8, 32, WIDE), (1024, 32, 16, WIDE), (2048, 16, 8, WIDE), (4096, 1, 4, WIDE), (100, 1, 40, NARROW),
])
def test_refreshed_rows(route, batch, heads, seq, want):
    assert route(batch, heads, seq, True, False, False) == want


def test_cut_keys_need_the_workspace_and_long_sequences(route):
    for seq, workspace, want in ((1920, 1, NARROW), (1921, 0, NARROW), (1921, 1, LAID_OUT), (4096, 1, LAID_OUT)):
        assert route(1, 32, seq, True, False, workspace) == want


@pytest.mark.parametrize("listed", [False, True])
def test_all_rows(route, listed):
    for batch, heads, seq, want in ((8, 32, 2048, TALL), (1, 32, 4096, TALL), (1, 32, 1024, WIDE), (2048, 16, 8, TALL)):
        assert route(batch, heads, seq, listed, listed, True) == want
