"""The rule that picks the tile shape of an all-row bf16 projection (csrc/gemm_route.h), evaluated
on the CPU over rows 1 .. 6000 and every hidden size in steps of 64 up to 8192, for the
projections that a layer and a model make from them.  The route that cuts k over two workgroups
owns a workspace of kSplitTiles tiles and as many counters: it must never get more, nor be
taken without a workspace, nor depend on how large a context was made."""
import os
import subprocess

import test_gpu_block as block
import test_gpu_kernels as kernels
import test_gpu_layer as layer
import test_gpu_model as model

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SWEEP = r"""
#include <cstdio>
#include "gemm_route.h"
using namespace dare;
static long bad;
static void fail(const char* what, int m, int n, int k) {
  if (bad++ < 10) std::printf("%s: m %d n %d k %d\n", what, m, n, k);
}
int main() {
  long split = 0;
  for (int d = 64; d <= 8192; d += 64)
    for (int m = 1; m <= 6000; ++m) {
      const int shapes[][2] = {{d, d}, {3 * d, d}, {d, 3 * d}, {d, 4 * d}, {6 * d, d}};  // n, k
      for (const auto& s : shapes) {
        const int n = s[0], k = s[1];
        const GemmRoute with = gemm_route(m, n, k, 1, true), without = gemm_route(m, n, k, 1, false);
        if (without == GemmRoute::kPp128Split) fail("no workspace", m, n, k);
        if (gemm_route(m, n, k, 2, true) == GemmRoute::kPp128Split) fail("k already in ranges", m, n, k);
        const int t = tiles_of(m, n, kPpRows, 128);
        // a round of 256 x 128 tiles takes 1.5 times one of 128 x 128
        if (without == GemmRoute::kPp128 && (t + 255) / 256 >= (tiles_of(m, n, 128, 128) + 255) / 256)
          fail("larger tiles in as many rounds", m, n, k);
        if (with != GemmRoute::kPp128Split) {
          if (with != without) fail("workspace changes another route", m, n, k);
          continue;
        }
        ++split;
        if (t > kSplitTiles) fail("more tiles than the workspace holds", m, n, k);
        if (k / kRouteBK % 2 || k / kRouteBK < kSplitMinSteps) fail("k cannot be cut", m, n, k);
        // a workspace exists in every context that holds this many rows or more
        for (int more = 0; more <= 4096; more += 512)
          if (!gemm_may_split(m + more, n, k)) fail("route without its workspace", m + more, n, k);
      }
    }
  std::printf("split %ld bad %ld\n", split, bad);
  return bad != 0;
}
"""


def _run(tmp_path, text):
    src, exe = tmp_path / "sweep.cpp", tmp_path / "sweep"
    src.write_text(text)
    subprocess.run(["g++", "-std=c++17", "-O2", "-I", os.path.join(ROOT, "paper_2605_08134_amd", "csrc"),
                    str(src), "-o", str(exe)], check=True)
    return subprocess.run([str(exe)], capture_output=True, text=True)


def test_cut_projection_never_exceeds_its_workspace(tmp_path):
    r = _run(tmp_path, SWEEP)
    assert r.returncode == 0, r.stdout
    assert int(r.stdout.split()[1]) > 1000     # the sweep does reach the route


SCORE_LDS = r"""
#include <cstdio>
#include "gemm_route.h"
using namespace dare;
int main() {
  int bad = 0;
  for (int width = 64; width <= 128; width += 64)
    for (int bm = 16; bm <= 64; bm *= 2) {
      const int at = score_arrived_offset(bm, width);
      for (int row = 0; row < bm; ++row)
        for (int col = 0; col < width; ++col) {
          const int q = (row * score_query_stride(width) + col) * 4;
          if (q < at + 4 && at < q + 4) ++bad;
        }
    }
  std::printf("%d\n", bad);
  return bad != 0;
}
"""


def test_last_flag_of_the_scored_columns_is_no_query_word(tmp_path):
    """Every wave of the last workgroup reads that it is the last and then writes its queries into
    the same LDS array, with no barrier in between: the two must not share a word."""
    assert _run(tmp_path, SCORE_LDS).returncode == 0


RANGES = r"""
#include <cstdio>
#include "gemm_route.h"
using namespace dare;
int main() {
  int bad = 0;
  const struct { int m, n, parts; GemmRoute want; } at[] = {
      {1024, 128, 8, GemmRoute::kTile64}, {4096, 128, 4, GemmRoute::kTile64},  // a round of either
      {8192, 128, 2, GemmRoute::kTile64}, {8193, 128, 2, GemmRoute::kTile128}, {9000, 128, 2, GemmRoute::kTile128},
      {16384, 128, 2, GemmRoute::kTile128}, {4096, 4096, 2, GemmRoute::kTile128}, {65, 8192, 8, GemmRoute::kTile128},
      {300, 4096, 4, GemmRoute::kTile64}, {9000, 192, 2, GemmRoute::kTile64}};
  for (const auto& c : at)
    for (int workspace = 0; workspace < 2; ++workspace)
        if (gemm_route(c.m, c.n, 4096, c.parts, workspace) != c.want) std::printf("%d x %d\n", c.m, c.n), ++bad;
  return bad != 0;
}
"""


def test_k_in_ranges_takes_large_tiles_where_they_need_fewer_rounds(tmp_path):
    r = _run(tmp_path, RANGES)
    assert r.returncode == 0, r.stdout


SPLIT = r"""
#include <cstdio>
#include "gemm_route.h"
using namespace dare;
int main() {
  int bad = 0;
  const struct { int m, n, k; bool want; } at[] = {
      {1024, 4096, 12288, true}, {600, 4096, 12288, true}, {768, 4096, 12288, true}, {768, 3072, 9216, true},
      {2305, 1024, 9216, true}, {2305, 1024, 6144, false},     // 128 x 96 otherwise: from 144 k-steps on
      {2048, 2048, 6144, true}, {1793, 2048, 6144, true},      // 128 x 128 otherwise: from 96
      {2048, 1024, 6144, false}, {1793, 1024, 6144, false}, {402, 4096, 12288, false},   // 64 x 128
      {2305, 2048, 6144, false}, {1025, 4096, 12288, false},   // more than the workspace holds
      {1024, 4096, 4096, false}};
  for (const auto& c : at)
    if ((gemm_route(c.m, c.n, c.k, 1, true) == GemmRoute::kPp128Split) != c.want)
      std::printf("%d x %d x %d\n", c.m, c.n, c.k), ++bad;
  return bad != 0;
}
"""


def test_which_projections_are_cut_over_two_workgroups(tmp_path):
    r = _run(tmp_path, SPLIT)
    assert r.returncode == 0, r.stdout


AHEAD = r"""
#include <cstdio>
#include "gemm_route.h"
using namespace dare;
int main() {
  int bad = 0;
  for (int n = 64; n <= 49152; n += 64)
    for (int wg = 8; wg <= 256; wg += 8) {
      const long per_xcd = (n + 7) / 8, once = wg / 8 * 16, loads = ahead_loads(n, wg);
      if (loads < 1 || loads > 8 || loads * once * 512 > 2 << 20) ++bad;      // bytes in the L2
      if (loads < 8 && loads * once < per_xcd) ++bad;                          // the whole share
      if (loads > 1 && (loads - 1) * once >= per_xcd) ++bad;                   // and no load that only repeats rows
    }
  std::printf("%d\n", bad);
  return bad != 0;
}
"""


def test_weights_read_ahead_cover_every_width(tmp_path):
    """Not only the two widths of one hidden size: the share of an XCD whole, up to half of its L2."""
    r = _run(tmp_path, AHEAD)
    assert r.returncode == 0, r.stdout


SHAPES = r"""
#include <cstdio>
#include "gemm_route.h"
using namespace dare;
int main() {
  const char* name[] = {"ranges 64 x 64", "ranges 128 x 128", "64 x 64", "64 x 96", "64 x 128", "128 x 48", "128 x 64", "128 x 96",
                        "128 x 128", "128 x 192", "256 x 128", "256 x 192", "256 x 256", "256 x 256 cut", "split",
                        "256 x 192 four waves", "256 x 256 four waves"};
  static_assert((int)GemmRoute::kQuad256 == 16, "a shape without a name");
  int listed, m, n, k;
  while (std::scanf("%d %d %d %d", &listed, &m, &n, &k) == 4)
    std::printf("%s\n", name[(int)(listed ? best_tile(m, n, true) : gemm_route(m, n, k, 1, false))]);
}
"""


def test_gpu_tests_reach_the_shapes_that_they_name(tmp_path):
    """The sizes of tests/test_gpu_kernels.py and test_gpu_block.py, asked of the rule on the CPU: each gets the tile shape
    that its text names, and between them they take every shape that all rows and that listed rows can get."""
    src, exe = tmp_path / "shapes.cpp", tmp_path / "shapes"
    src.write_text(SHAPES)
    subprocess.run(["g++", "-std=c++17", "-I", os.path.join(ROOT, "paper_2605_08134_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True)
    want = {size: kernels.EVERY_TILE[size[:3]] for size in kernels.EVERY_TILE_SIZES}
    for m, n, k, _, text in kernels.LARGE_TILES:
        want[False, m, n, k] = text.split(",")[0]
    for m, seg, k, _, text in block.ROPE_TILES:      # (their lists have a length that the host knows)
        want[False, m, 3 * seg, k] = text
    m, seg, k, text = block.STREAM_TILE
    want[False, m, 3 * seg, k] = text
    (b, t, d, f), text = model.GATE_PAST_THE_L2
    want[False, b * t, 2 * f, d] = text
    for n, count, text in kernels.LONG_K_TILES:
        if text.startswith("stream"):
            assert count <= 32 and n < 8192
        else:
            want[True, count, n, 4096] = text.split(",")[0]
    ask = "".join("%d %d %d %d\n" % size for size in want)
    got = subprocess.run([str(exe)], input=ask, capture_output=True, text=True, check=True).stdout.splitlines()
    assert dict(zip(want, got)) == want
    large = {"128 x 96", "128 x 128", "128 x 192", "256 x 128", "256 x 192", "256 x 256"}
    assert {want[s] for s in want if not s[0]} == {"64 x 64", "64 x 96", "64 x 128", "256 x 192 four waves",
                                                   "256 x 256 four waves"} | large
    assert {want[s] for s in want if s[0]} == {"64 x 64", "128 x 48", "128 x 64", "256 x 256 cut"} | large


FORMS = r"""
#include <cstdio>
#include "gemm_route.h"
using namespace dare;
int main() {
  long bad = 0, four = 0, eight = 0;
  const struct { int m, n, k; GemmRoute want; } at[] = {
      {1024, 12288, 4096, GemmRoute::kPp192}, {640, 12288, 4096, GemmRoute::kPp192}, {3600, 3072, 1024, GemmRoute::kPp192},   // one round
      {1024, 24576, 4096, GemmRoute::kQuad192}, {1536, 12288, 4096, GemmRoute::kQuad192},                                     // two
      {1536, 9216, 3072, GemmRoute::kPp256}, {2560, 6144, 2048, GemmRoute::kPp256}, {5120, 3072, 1024, GemmRoute::kPp256},
      {7000, 2048, 2048, GemmRoute::kQuad256}, {4096, 4096, 4096, GemmRoute::kQuad256}, {4096, 24576, 4096, GemmRoute::kQuad256}};
  for (const auto& c : at)
    if (gemm_route(c.m, c.n, c.k, 1, false) != c.want) std::printf("%d x %d x %d\n", c.m, c.n, c.k), ++bad;
  for (int n = 64; n <= 32768; n += 192)
    for (int m = 1; m <= 40000; m = m < 600 ? m + 13 : m + 397)
      for (int k = 64; k <= 12288; k *= 2) {
        const GemmRoute r = gemm_route(m, n, k, 1, false), shape = best_tile(m, n, false);
        const bool q192 = r == GemmRoute::kQuad192, q256 = r == GemmRoute::kQuad256;
        if ((q192 ? GemmRoute::kPp192 : q256 ? GemmRoute::kPp256 : r) != shape) ++bad;                          // the form alone
        const bool one = tiles_of(m, n, kPpRows, shape == GemmRoute::kPp192 ? 192 : 256) <= 256;
        if (q192 && one) ++bad;
        if ((q192 || q256) && k < 192) ++bad;
        if ((shape == GemmRoute::kPp192 || shape == GemmRoute::kPp256) && !one && k >= 192 && !q192 && !q256) ++bad;
        four += q192 || q256;
        eight += r == GemmRoute::kPp192 || r == GemmRoute::kPp256;
      }
  std::printf("four %ld eight %ld bad %ld\n", four, eight, bad);
  return bad != 0 || four < 1000 || eight < 1000;
}
"""


def test_one_round_of_large_tiles_keeps_eight_waves(tmp_path):
    r = _run(tmp_path, FORMS)
    assert r.returncode == 0, r.stdout


PART = r"""
#include <cstdio>
#include "gemm_route.h"
using namespace dare;
int main() {
  long bad = 0, later = 0;
  // refreshed in per cent; both ways were measured at the first ones, and differ by 2 % or more
  const struct { int m, percent, d; bool want; } at[] = {
      {1500, 50, 4096, true}, {1500, 80, 4096, false}, {2048, 5, 4096, false}, {2048, 50, 4096, false}, {2331, 25, 4096, true},
      {2331, 50, 4096, false}, {2560, 25, 4096, true}, {2560, 50, 4096, false}, {3200, 50, 4096, true}, {3200, 80, 4096, false},
      {4096, 5, 4096, true}, {4096, 25, 4096, false}, {5120, 25, 4096, true}, {5120, 50, 4096, false}, {16384, 50, 4096, true},
      {16384, 80, 4096, false}, {2800, 80, 2048, true}, {2800, 100, 2048, false}, {8192, 5, 2048, true}, {8192, 60, 2048, false},
      {5600, 50, 1024, true}, {6000, 35, 3072, true}, {2048, 65, 3072, false}, {1700, 25, 4096, true}, {1700, 35, 4096, false},
      {1 << 29, 50, 64, false}, {1 << 29, 50, 4096, false}, {600, 5, 4096, false}, {1024, 5, 4096, false}, {1023, 0, 8192, false},
      {4096, 50, 512, false}, {4096, 50, 128, false}};
  for (const auto& c : at)
    if (queries_of_listed_rows(c.m, (long)c.m * c.percent / 100, c.d) != c.want) std::printf("%d x %d, %d\n", c.m, c.d, c.percent), ++bad;
  for (int d = 64; d <= 8192; d += 64)
    for (int m = 1; m <= 40000; m = m < 600 ? m + 13 : m + 397) {
      if (queries_of_listed_rows(m, m, d)) ++bad;      // where every query is read there is nothing to save
      if (queries_of_listed_rows(m, m / 2, d)) {
        ++later;
        if (m < kPartMinRows || d / kRouteBK < kQuadMinSteps) ++bad;
        if (!queries_of_listed_rows(m, m / 4, d)) ++bad;      // fewer save no less
      }
      for (int part = 0; part <= m; part += m / 3 + 1) {
        const int tn = part_columns(m, 3 * d, part, d);
        for (int o = 3; o <= 4; ++o)
          if (tn < 3 || tn > 4 || quad_cost(part_tiles(m, 3 * d, part, d, o), o) < quad_cost(part_tiles(m, 3 * d, part, d, tn), tn)) ++bad;
      }
    }
  std::printf("later %ld bad %ld\n", later, bad);
  return bad != 0;
}
"""


def test_queries_behind_the_score_where_they_save_rounds(tmp_path):
    r = _run(tmp_path, PART)
    assert r.returncode == 0, r.stdout


WIDTHS = r"""
#include <cstdio>
#include "gemm_route.h"
int main() {
  int m, d, part;
  while (std::scanf("%d %d %d", &m, &d, &part) == 3) std::printf("%d\n", dare::part_columns(m, 3 * d, part, d));
}
"""


def test_gpu_tests_reach_both_widths_of_the_joint_launch(tmp_path):
    src, exe = tmp_path / "widths.cpp", tmp_path / "widths"
    src.write_text(WIDTHS)
    subprocess.run(["g++", "-std=c++17", "-I", os.path.join(ROOT, "paper_2605_08134_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True)
    for batch, seq, hidden, _ in layer.QUERIES_LATER:
        counts = (batch * seq, batch * seq // 5, batch * seq // 3, 1, 0)
        ask = "".join("%d %d %d\n" % (batch * seq, hidden, n) for n in counts)
        got = subprocess.run([str(exe)], input=ask, capture_output=True, text=True, check=True).stdout.split()
        assert set(got) == {"3", "4"}, (batch, seq, hidden, got)


LATER = r"""
#include <cstdio>
#include "gemm_route.h"
int main() {
  int m, d, refreshed;
  while (std::scanf("%d %d %d", &m, &d, &refreshed) == 3) std::printf("%d\n", dare::queries_of_listed_rows(m, refreshed, d));
}
"""


def test_gpu_tests_reach_the_queries_behind_the_score(tmp_path):
    src, exe = tmp_path / "later.cpp", tmp_path / "later"
    src.write_text(LATER)
    subprocess.run(["g++", "-std=c++17", "-I", os.path.join(ROOT, "paper_2605_08134_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True)
    want = {(b * t, d, b * t // 2): "1" for b, t, d, _ in layer.QUERIES_LATER}
    b, t, d = layer.BY_RATE
    want.update({(b * t, d, b * t // 2): "0", (b * t, d, b * t // 4): "1", (1500, 4096, 750): "1"})
    ask = "".join("%d %d %d\n" % size for size in want)
    got = subprocess.run([str(exe)], input=ask, capture_output=True, text=True, check=True).stdout.split()
    assert dict(zip(want, got)) == want


LISTED = r"""
#include <cstdio>
#include "gemm_route.h"
using namespace dare;
// the cost again in 64 bits
static long cost(long m, long n, long bm, long bn, long full, long again) {
  const long tiles = (m + bm - 1) / bm * ((n + bn - 1) / bn), rounds = (tiles + 255) / 256;
  return (rounds > 1 ? again : full) * (rounds * 256 + tiles);
}
int main() {
  long bad = 0, cut = 0;
  for (int n = 64; n <= 1 << 21; n = n < 32768 ? n + 64 : n * 2 + 64)
    for (int m = 1; m <= 1 << 20; m = m < 400 ? m + 1 : (m < 20000 ? m + 97 : m * 2 + 1)) {
      const GemmRoute r = best_tile(m, n, true);
      const long t4 = (m + 255l) / 256 * ((n + 255l) / 256);
      if (r == GemmRoute::kTile64 || r == GemmRoute::kTile128 || r == GemmRoute::k64x96 || r == GemmRoute::k64x128 ||
          r == GemmRoute::kPp128Split) ++bad;                                            // no such shape in the kernel
      if (t4 > 8192) continue;
      if (cost(m, n, 64, 64, 153, 229) != tile_cost(m, n, 64, 64, 153, 229) ||
          cost(m, n, 128, 48, 210, 273) != tile_cost(m, n, 128, 48, 210, 273) ||
          cost(m, n, 256, 256, 1460, 1460) != tile_cost(m, n, 256, 256, 1460, 1460)) ++bad;   // 32 bits hold it
      if (r != GemmRoute::kPp256Cut) continue;
      ++cut;
      if (n % 256 || t4 <= 256 || t4 % 256 == 0 || t4 % 256 > 128) ++bad;                // whole rounds in front of the cut one
    }
  std::printf("cut %ld bad %ld\n", cut, bad);
  return bad != 0;
}
"""


def test_listed_rows_over_the_whole_range(tmp_path):
    """The rule as the kernel evaluates it, up to a million rows and two million columns."""
    r = _run(tmp_path, LISTED)
    assert r.returncode == 0, r.stdout
    assert int(r.stdout.split()[1]) > 1000
