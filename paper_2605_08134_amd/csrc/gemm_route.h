// Tile shape of a bf16 projection whose row count the host knows, as plain host arithmetic: no HIP
// here, so that the rule can be evaluated over its whole range without a GPU.
#pragma once

namespace dare {

enum class GemmRoute {
  kTile64,      // 64 x 64, four waves
  kTile128,     // 128 x 128 on the 16-wide MFMA shape, eight waves
  kRows64,      // 64 x 128 on the 16-wide MFMA shape: one row tile
  kRows128,     // 128 x 128 on the 16-wide MFMA shape: one row tile
  kPp128,       // ping-pong tiles of 256 rows x 128, 192, 256 columns
  kPp192,
  kPp256,
  kPp128Split,  // 256 x 128, two workgroups on the halves of a tile's k; needs the workspace
};

constexpr int kRouteBK = 64;        // k per k-step
constexpr int kPpRows = 256;        // rows of a ping-pong tile
constexpr int kSplitTiles = 128;    // tiles the workspace holds: two workgroups each fill the 256 CUs once
// k-steps of a tile whose k is cut.  The hand-over costs about 5 us and 33 MB written past L2: 1024 x 4096
// outputs with 64 k-steps gain nothing (a dense layer step 156.4 us with and 157.1 without, a K/V reuse step
// 173.4 and 172.8), 192 k-steps 25 us of 122; the two time lines cross near 55.
constexpr int kSplitMinSteps = 96;

constexpr int tiles_of(int m, int n, int bm, int bn) { return ((m + bm - 1) / bm) * ((n + bn - 1) / bn); }

// Whether some projection of at most m rows with this n and k takes the route that needs the workspace
constexpr bool gemm_may_split(long m, long n, long k) {
  return (m + kPpRows - 1) / kPpRows * ((n + 127) / 128) >= kSplitTiles / 2 && k / kRouteBK % 2 == 0 &&
         k / kRouteBK >= kSplitMinSteps;
}

// Once 256-row tiles fill most of the chip, the ping-pong tile
// wins: 256 x 192 costs about 3/4 of 256 x 256 (1870 against 2500 cycles per k-step), so the narrow
// one is taken where it needs fewer quarter-rounds of the 256 CUs (1024 x 12288: one full round
// against one round with 64 CUs idle, 78 against 85 us; 2331 x 12288: three against two, 209 against
// 198 us).  256 x 128 takes over while it fills more than half of the CUs and needs fewer rounds of
// them than 128 x 128 (a round at k = 4096 takes 59 us against 39: 520 x 6144, 144 tiles against 240, one
// round each; 600 x 12288, 288 against 480, two each: 96 against 83 us; 1024 x 9216 x 3072, two against
// three: 78 against 94), and with two workgroups
// per tile where there are kSplitTiles / 2 to kSplitTiles of them.  128 x 128 with 8 waves is the best
// shape when the larger ones would leave most CUs idle.
// One row tile (the output embedding of a few rows): a stream over the weights, of which 256-row
// tiles pull as many bytes of repeated rows as of weights.  64 and 128 rows with the 16-wide MFMA
// shape and as many weight rows in flight as fit (us, before in 256-row tiles; 1.04 GB of weights,
// k = 4096): 32 x 126464 229 -> 174 (5.9 TB/s), 64 x 126464 243 -> 205, 128 x 126464 244 -> 220,
// 128 x 24576 40 (128 x 128 tiles, 32-wide) -> 37.
constexpr GemmRoute gemm_route(int m, int n, int k, int k_parts, bool workspace) {
  const int t128 = tiles_of(m, n, 128, 128);
  if (k_parts <= 1 && m <= 64 && tiles_of(m, n, 64, 128) >= 192) return GemmRoute::kRows64;
  if (k_parts <= 1 && m > 64 && m <= 128 && t128 >= 64) return GemmRoute::kRows128;
  if (k_parts <= 1 && m > 128) {
    const int t3 = tiles_of(m, n, kPpRows, 192), t4 = tiles_of(m, n, kPpRows, 256);
    const int q3 = 3 * ((t3 + 255) / 256), q4 = 4 * ((t4 + 255) / 256);
    if (t3 >= 224 && (q3 < q4 || t4 < 176)) return GemmRoute::kPp192;
    if (t4 >= 176) return GemmRoute::kPp256;
    const int t2 = tiles_of(m, n, kPpRows, 128), ksteps = k / kRouteBK;
    if (t2 > kSplitTiles && (t2 + 255) / 256 < (t128 + 255) / 256) return GemmRoute::kPp128;
    if (workspace && t2 >= kSplitTiles / 2 && t2 <= kSplitTiles && ksteps % 2 == 0 && ksteps >= kSplitMinSteps)
      return GemmRoute::kPp128Split;
  }
  if (k_parts <= 1 && m > 64 && n % 128 == 0 && t128 >= 64) return GemmRoute::kTile128;
  return GemmRoute::kTile64;
}

// Scored columns: whether the score is taken in the launch that projects them, rather than in one of its
// own.  With a long k and one round of 64 x 64 tiles or a little less, the tiles of the plain projection
// pull less per CU than whole queries do (projection, score and selection of a step that refreshes
// nothing, k = 4096, one launch against two: 1024 rows 18.0 and 18.3 us, 2048 21.0 and 20.9, 3072 27.0 and 25.9, 4096 27.7 and
// 25.5, 6144 35.2 and 32.9, 8192, where the plain projection takes larger tiles, 35.9 and 50.9; k = 2048:
// 4096 rows 22.0 and 22.9).
constexpr bool score_in_projection(int rows, int k) { return k < 3072 || rows <= 2560 || rows > 8064; }

// LDS of the scored-column projection once its k loop is over: bm queries, score_query_stride floats
// apart, from offset 0, and the word that says whether the workgroup is the last one
constexpr int score_query_stride(int width) { return width + 4; }
constexpr int score_arrived_offset(int bm, int width) { return bm * score_query_stride(width) * 4; }

}  // namespace dare
