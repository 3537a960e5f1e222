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
  std::printf("%d", (int)dare::attn_route(atol(a[1]), atol(a[2]), atoi(a[3]), atoi(a[4]), atoi(a[5]), atoi(a[6]), atoi(a[7]), atoi(a[8])));
}
"""
NARROW, WIDE, TALL, LAID_OUT = range(4)


@pytest.fixture(scope="module")
def route(tmp_path_factory):
    d = tmp_path_factory.mktemp("attn_route")
    (d / "probe.cpp").write_text(PROBE)
    subprocess.run(["g++", "-std=c++17", "-I", os.path.join(ROOT, "paper_2605_08134_amd", "csrc"), str(d / "probe.cpp"),
                    "-o", str(d / "probe")], check=True)
    return lambda *args, dh=128, active=0: int(subprocess.run([str(d / "probe")] + [str(int(v)) for v in (*args, dh, active)],
                                                              capture_output=True, text=True, check=True).stdout)


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
        assert route(batch, heads, seq, listed, listed, True, dh=64) == want
    for dh, want in ((128, TALL), (64, WIDE)):   # 288 blocks of 128 rows, 160 of 256
        assert route(1, 32, 1152, listed, listed, True, dh=dh) == want


@pytest.mark.parametrize("batch,heads,seq,active,want", [
    (1, 32, 1536, 1024, WIDE), (1, 32, 1536, 1025, TALL), (1, 32, 1536, 0, TALL), (2, 32, 700, 444, WIDE),
    (1, 16, 2560, 1792, WIDE), (1, 32, 1792, 892, WIDE), (1, 32, 4096, 596, WIDE), (4, 32, 4096, 2048, TALL),
    (8, 16, 300, 256, WIDE), (8, 16, 300, 257, TALL), (17, 16, 40, 30, TALL),
])
def test_all_rows_behind_a_frozen_prefix_count_without_it(route, batch, heads, seq, active, want):
    assert route(batch, heads, seq, True, True, True, active=active) == want


SECOND = r"""
#include <initializer_list>
#include "attn_route.h"
using namespace dare;
int main() {
  for (int batch = 1; batch <= 300; batch += batch < 20 ? 1 : 7)
    for (int heads : {1, 4, 8, 16, 24, 32, 64})
      for (int rows = 1; rows <= 4200; rows += 1 + rows / 37) {
        const long b128 = (long)batch * heads * ((rows + 127) / 128), b256 = (long)batch * heads * ((rows + 255) / 256);
        const bool tall = attn_route(batch, heads, 4200, true, true, true, 128, rows) == AttnRoute::kTall;
        if (tall != (b128 > 256) || attn_second_reference((long)batch * heads, rows) != (b256 < 256)) return 1;
        // heads of 64 have no second reference: two key-waves wherever the rule asks for one
        if (attn_second_reference((long)batch * heads, rows) && attn_route(batch, heads, 4200, true, true, true, 64, rows) == AttnRoute::kTall) return 2;
      }
  return 0;
}
"""


def test_a_second_reference_where_two_key_waves_were_the_other_choice(tmp_path):
    (tmp_path / "second.cpp").write_text(SECOND)
    subprocess.run(["g++", "-std=c++17", "-I", os.path.join(ROOT, "paper_2605_08134_amd", "csrc"), str(tmp_path / "second.cpp"),
                    "-o", str(tmp_path / "second")], check=True)
    assert subprocess.run([str(tmp_path / "second")]).returncode == 0


PLACES = r"""
#include <cstdio>
#include <vector>
#include "attn_route.h"
using namespace dare;
int main() {
  int bad = 0;
  for (int per_xcd = 1; per_xcd <= 40; ++per_xcd)
    for (int n_blocks = 1; n_blocks <= 9; ++n_blocks)
      for (int turn : {1, attn_turn(8 * per_xcd, true, false)}) {
        std::vector<int> at(per_xcd * n_blocks, -1);
        for (int slot = 0; slot < per_xcd * n_blocks; ++slot) {
          const AttnPlace x = attn_place(slot, per_xcd, n_blocks, turn);
          if (x.pair >= (unsigned)per_xcd || x.block >= (unsigned)n_blocks || at[x.pair * n_blocks + x.block] >= 0) ++bad;
          else at[x.pair * n_blocks + x.block] = slot;
        }
        for (int i = 0; i < per_xcd * n_blocks; ++i) {
          if (i % n_blocks && at[i] - at[i - 1] != (turn == 1 ? 1 : turn < per_xcd - i / n_blocks / turn * turn ? turn : per_xcd - i / n_blocks / turn * turn)) ++bad;
        }
      }
  std::printf("%d\n", bad);
  return bad != 0;
}
"""


def test_every_block_has_one_workgroup_and_follows_its_pairs_last_one(tmp_path):
    """Over all counts of pairs and blocks: each block once, and a pair's next block at most eight workgroups of
    the XCD behind its last one, however many pairs there are (its keys and values are in the L2 then)."""
    (tmp_path / "places.cpp").write_text(PLACES)
    subprocess.run(["g++", "-std=c++17", "-I", os.path.join(ROOT, "paper_2605_08134_amd", "csrc"),
                    str(tmp_path / "places.cpp"), "-o", str(tmp_path / "places")], check=True)
    r = subprocess.run([str(tmp_path / "places")], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


TURN = r"""
#include <cstdio>
#include <cstdlib>
#include "attn_route.h"
int main(int, char** a) {
  std::printf("%d %d", dare::attn_turn(atoi(a[1]), atoi(a[2]), atoi(a[3])), dare::attn_at_once(atoi(a[1]), atoi(a[4]), atoi(a[5])));
}
"""


def test_turns_and_readers_ahead(tmp_path):
    (tmp_path / "turn.cpp").write_text(TURN)
    subprocess.run(["g++", "-std=c++17", "-I", os.path.join(ROOT, "paper_2605_08134_amd", "csrc"),
                    str(tmp_path / "turn.cpp"), "-o", str(tmp_path / "turn")], check=True)
    for (pairs, listed, many, seq, dh), want in {
        (32, 1, 0, 1024, 128): (4, 8), (32, 1, 1, 1024, 128): (1, 8), (32, 0, 0, 1024, 128): (1, 8),
        (2048, 1, 0, 512, 128): (8, 0),    # no CU for a reader
        (8, 1, 0, 201, 128): (1, 0),       # two key steps
        (60, 1, 0, 1100, 128): (8, 0), (60, 1, 0, 1024, 128): (8, 4), (60, 1, 0, 1024, 64): (8, 8),   # 4 MB of L2
    }.items():
        r = subprocess.run([str(tmp_path / "turn")] + [str(v) for v in (pairs, listed, many, seq, dh)],
                           capture_output=True, text=True, check=True)
        assert tuple(map(int, r.stdout.split())) == want, (pairs, seq, dh)


HALVES = r"""
#include <cstdio>
#include <vector>
#include "attn_route.h"
int main() {
  for (int slots : {1, 7, 32, 64})
    for (int n = 0; n < 400; ++n) {
      const int whole = dare::attn_whole_blocks(n, slots, true), end = 2 * n - whole;
      if (dare::attn_whole_blocks(n, slots, false) != n || whole > n || (whole < n && (whole % slots || end - whole > slots))) return 1;
      std::vector<int> rows(2 * n);  // halves of blocks, as the kernel numbers them
      for (int s = 0; s < end; ++s)
        if (s < whole) ++rows[2 * s], ++rows[2 * s + 1]; else ++rows[2 * (whole + (s - whole) / 2) + (s - whole) % 2];
      for (int r : rows) if (r != 1) return 2;
    }
  return 0;
}
"""


def test_every_block_of_128_rows_runs_whole_or_in_two_halves(tmp_path):
    (tmp_path / "halves.cpp").write_text(HALVES)
    subprocess.run(["g++", "-std=c++17", "-I", os.path.join(ROOT, "paper_2605_08134_amd", "csrc"), str(tmp_path / "halves.cpp"),
                    "-o", str(tmp_path / "halves")], check=True)
    assert subprocess.run([str(tmp_path / "halves")]).returncode == 0
