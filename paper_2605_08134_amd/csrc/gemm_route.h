// Tile shape of a bf16 projection, as plain host arithmetic: no HIP here, so that the rule can be
// evaluated over its whole range without a GPU.  Where the row count is known on the device only, the kernel
// evaluates the same rule.
#pragma once

namespace dare {

enum class GemmRoute {
  kTile64,      // k in ranges: 64 x 64, four waves
  kTile128,     // k in ranges: 128 x 128, eight waves
  k64x64,       // eight waves, 16-wide MFMA shape
  k64x96,
  k64x128,
  k128x48,
  k128x64,
  k128x96,
  k128x128,
  k128x192,
  kPp128,       // 256 rows x 128, 192, 256 columns: ping-pong tiles (eight waves)
  kPp192,
  kPp256,
  kPp256Cut,    // the last round of 256 x 256 cut into 128 x 128 (listed rows)
  kPp128Split,  // 256 x 128, two workgroups on the halves of a tile's k; needs the workspace
  kQuad192,     // 256 rows x 192, 256 columns: four waves, one pipeline over a workgroup's tiles (all rows)
  kQuad256,
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

// What a projection takes in tiles of bm x bn, in units that the shapes share (with 64 k-steps 512000 are about 70
// us; the k-steps are common to all shapes and drop out).  A round in which all 256 CUs have a tile counts 512
// times `full`, and idle CUs save half of their share of it (power, and the operands from beyond the L2, are
// shared by those that work).  In several rounds it is `again` instead of `full`: nothing hides the ends of the
// 16-wide loop's shapes, and small ones pull the weights again for every row of tiles (300 x 12288 x 4096: 64 x 64 73
// us, 256 x 128 52).
// Fitted to 120 products of 40 to 16384 rows by 512 to 24576 columns, k from 512 to 12288, in every shape with eight waves: the
// shape chosen is within 3 % of the fastest one of those (several rounds of 256 x 192 and 256 of all rows have four and take 9 and 12 % less,
// which the choice does not count) but for 1300 x 4096 x 12288 (10 %: 192 x 128, which nothing else
// wants) and 256 x 24576 x 4096 (10 %).  A rule by
// thresholds on tile counts, made for 1024 tokens of 4096, was off by up to 2 (us, before and now, the loop of gemm_tile16
// included: 402 x 2048 x 2048 20.6 and 9.6, 256 x 4096 x 4096 34.1 and 16.6, 1000 x 9216 x 3072 75.9 and 50.2, 2331 x 4096 x
// 4096 97 and 69; refreshed rows, 1300 x 4096 x 4096 75 and 52, 2870 x 4096 x 4096 124 and 82, 4096 x 4096 x 4096 166 and 97,
// 600 x 12288 x 4096 80 and 65).
// (Whole numbers: the device evaluates it on its scalar unit.)
constexpr int tile_cost(int m, int n, int bm, int bn, int full, int again) {
  const int tiles = tiles_of(m, n, bm, bn), rounds = (tiles + 255) >> 8;
  return (rounds > 1 ? again : full) * (rounds * 256 + tiles);
}

// The shape for m rows and n columns.  listed: rows read through a list, which prefers many rows to many columns
// in a small tile (128 x 64 against 64 x 128: 400 x 4096 28.0 and 29.3 us, all rows 23.1 and 21.5; 128 x 48 against 64 x
// 96: 250 x 6144 x 2048 13.6 and 14.0, 100 x 12288 x 4096 30.2 and 32.4).
// One round of the smallest tiles is the best wherever it is enough, and known without the rest (0.3 us on
// the device).
// (In line: called, the kernel gets the shape in a vector register and takes every branch on it, and all that lies
// behind, under lane masks.)
__attribute__((always_inline)) constexpr GemmRoute best_tile(int m, int n, bool listed) {
  if (tiles_of(m, n, 64, 64) <= 256) return GemmRoute::k64x64;
  if (tiles_of(m, n, kPpRows, 256) > 8192) return GemmRoute::kPp256;  // (and the costs below stay in 32 bits)
  GemmRoute best = GemmRoute::k64x64;
  int least = tile_cost(m, n, 64, 64, 153, 229);
  auto offer = [&](GemmRoute r, int cost) {
    if (cost < least) {
      least = cost;
      best = r;
    }
  };
  if (listed) {
    offer(GemmRoute::k128x48, tile_cost(m, n, 128, 48, 210, 273));
    offer(GemmRoute::k128x64, tile_cost(m, n, 128, 64, 245, 318));
  } else {
    offer(GemmRoute::k64x96, tile_cost(m, n, 64, 96, 235, 306));
    offer(GemmRoute::k64x128, tile_cost(m, n, 64, 128, 280, 364));
  }
  offer(GemmRoute::k128x96, tile_cost(m, n, 128, 96, 390, 448));
  offer(GemmRoute::k128x128, tile_cost(m, n, 128, 128, 490, 564));
  offer(GemmRoute::k128x192, tile_cost(m, n, 128, 192, 780, 897));
  offer(GemmRoute::kPp128, tile_cost(m, n, kPpRows, 128, 800, 848));
  offer(GemmRoute::kPp192, tile_cost(m, n, kPpRows, 192, 1150, 1150));
  offer(GemmRoute::kPp256, tile_cost(m, n, kPpRows, 256, 1460, 1460));
  const int t4 = tiles_of(m, n, kPpRows, 256), rest = t4 % 256;
  // (3266 x 12288 x 4096, 624 tiles of 256 x 256: 286 us, uncut 299)
  if (listed && n % 256 == 0 && t4 > 256 && rest > 0 && rest <= 128)
    offer(GemmRoute::kPp256Cut, 1460 * 512 * (t4 / 256) + tile_cost(4 * rest * 128, 128, 128, 128, 490, 490));
  return best;
}

// All rows in tiles of 256 x 192 or 256: four waves (gemm_tiles_quad) instead of eight.  They gain where a workgroup walks several
// tiles; a launch of one round has only their longer start (us of a layer or block step, eight waves and four, weights from memory:
// 1024 x 12288 x 4096 144.0 145.4, 640 x 12288 x 4096 121 126, 1320 x 6144 x 2048 84.6 88.0, 3600 x 3072 x 1024 65.2 67.0; two rounds,
// 4096 x 6144 x 2048 156.2 154.0, 1024 x 24576 x 4096 412 408, 1536 x 12288 x 4096 224 224; three, 3000 x 12288 x 4096 368 361).  In a
// round of 256 x 256 the k loop makes up for it with 64 k-steps and more, or with 32 where the weights, which come from memory, are
// the smaller operand (3600 x 4096 x 4096 425 420, 5120 x 3072 x 3072 351 346, 8192 x 2048 x 2048 277 275, 7000 x 2048 x 2048 256 255, but 1536 x
// 9216 x 3072 142.5 144.3, 2560 x 6144 x 2048 126.9 128.2, 5120 x 3072 x 1024 90.8 92.4).
// Not for one and two k-steps, less than the pipeline is long.
constexpr int kQuadMinSteps = 3;
constexpr bool four_waves(int m, int n, int k, int columns) {
  if (k / kRouteBK < kQuadMinSteps) return false;
  if (tiles_of(m, n, kPpRows, columns) > 256) return true;
  return columns == 256 && (k >= 4096 || (k >= 2048 && n <= 2 * m));
}

// Row count known on the host.  With the workspace, two workgroups per tile of 256 x 128 instead of 128 x 128 tiles where
// there are kSplitTiles / 2 to kSplitTiles of them and a long k: half of the tile's cost and the hand-over (1024 x 4096 x
// 12288: 97 against 112 us).  Instead of 128 x 96 from 144 k-steps on, where the 16-wide loop
// falls behind its cost (model steps of two layers, without and with: 768 x 3072 x 9216 431 and 412 us, 833 x 3072 x 9216 482 and
// 470, 1089 x 2048 x 12288 512 and 486, 2304 x 1024 x 12288 541 and 520, 512 x 6144 x 12288 720 and 699; with 96 to 128 k-steps
// 1089 x 2048 x 6144 319 and 326, 2240 x 1024 x 8192 379 and 396, 577 x 4096 x 8192 436 and 426).  64 x 128 stays (2048 x 1024 x
// 12288 431, cut 480).
constexpr GemmRoute gemm_route(int m, int n, int k, int k_parts, bool workspace) {
  if (k_parts > 1) {
    // A round of 128 x 128, one per CU, takes half as long again as one of 64 x 64, two per CU (us, 128 and 64: 8064 x 128 x
    // 4096 in two ranges 20.2 and 20.4, 9000 x 128 23.6 and 26.4, 16384 x 128 28.8 and 35.6, 4096 x 4096 194 and 246; 300 x
    // 4096 x 4096 in four 29.3 and 26.2)
    const long big = (long)tiles_of(m, n, 128, 128) * k_parts, small = (long)tiles_of(m, n, 64, 64) * k_parts;
    return n % 128 == 0 && 3 * ((big + 255) / 256) < 2 * ((small + 511) / 512) ? GemmRoute::kTile128 : GemmRoute::kTile64;
  }
  const GemmRoute best = best_tile(m, n, false);
  const int t2 = tiles_of(m, n, kPpRows, 128), ksteps = k / kRouteBK;
  if (workspace && t2 >= kSplitTiles / 2 && t2 <= kSplitTiles && ksteps % 2 == 0 && ksteps >= kSplitMinSteps &&
      (best == GemmRoute::k128x128 || (best == GemmRoute::k128x96 && ksteps >= 144)))
    return GemmRoute::kPp128Split;
  if (best == GemmRoute::kPp192 && four_waves(m, n, k, 192)) return GemmRoute::kQuad192;
  if (best == GemmRoute::kPp256 && four_waves(m, n, k, 256)) return GemmRoute::kQuad256;
  return best;
}

// What `tiles` tiles of 256 rows x 64 tn columns, tn 3 or 4, take in the four-wave form, in tile_cost's units (64 k-steps, one
// full round: 74 and 90 us).
constexpr long quad_cost(long tiles, int tn) {
  const long rounds = (tiles + 255) / 256;
  return (tn == 3 ? 1050 : 1290) * (rounds * 256 + tiles);
}

// Columns [0, part_n) for part_m listed rows and [part_n, n) for all m rows in one launch: its tiles, and the width
// (in 64 columns) of the least cost
constexpr long part_tiles(int m, int n, int part_m, int part_n, int tn) {
  return (long)tiles_of(m, n - part_n, kPpRows, 64 * tn) + tiles_of(part_m, part_n, kPpRows, 64 * tn);
}
__attribute__((always_inline)) constexpr int part_columns(int m, int n, int part_m, int part_n) {
  return quad_cost(part_tiles(m, n, part_m, part_n, 3), 3) < quad_cost(part_tiles(m, n, part_m, part_n, 4), 4) ? 3 : 4;
}

// What a launch of `tiles` tiles takes where it is compared with one of another number of tiles: rounds of the CUs above all, idle CUs
// in a round save a quarter of their share.  `full` as in tile_cost.
constexpr long rounds_cost(long tiles, int full) { return full * ((tiles + 255) / 256 * 768 + tiles) / 2; }

// Output reuse (mode O): queries for the refreshed rows only, with K and V of all rows in one launch, instead of Q, K and V of all
// rows.  The score then has its own pass over the hidden states, 5 us and 4 ns per row and 4096 of k more than what it takes as a
// by-product (27 us against 5 at 3200 x 4096), so the launch has to save a round, or most of one; below 1024 rows there is only one.
// refreshed: their number, known under a reuse rate; half of the rows where the score decides, so that no share up to a half loses.
// Block steps, 5, 25, 50 and 80 % refreshed, Q of all rows and behind the score (us): 1 x 1500 of 4096 219 185, 233 201, 260 233, 290 311;
// 4 x 800 353 284, 368 314, 409 383, 435 465; 8 x 2048 1372 1115, 1563 1351, 1833 1727, 2150 2224; 4 x 700 of 2048 140 115, 145 127, 153
// 138, 174 161; 4 x 1400 of 1024 103 88, 114 104, 125 116, 143 136.  Only where the rate says so: 3 x 777 of 4096 268 247, 282 266, 313 322,
// 326 342; 5 x 1024 477 401, 523 472, 557 582, 625 656.  Never: 1 x 2048 231 245, 251 267, 271 286, 316 335; 1 x 1024 145 163, 145 162, 154
// 172, 173 202.  47 sizes with six or eight shares, 330 steps: at the number that is refreshed the rule takes the slower way in
// 11, by 6 % once and else by 3 % or less; at half of the rows no step with up to a half loses, and with 80 % and all refreshed, where the
// score's pass saves nothing, the sizes that it takes lose 1 to 7 %, two of them 11 % (1 x 3000 of 4096, all, 497 556).
constexpr int kPartMinRows = 1024;
constexpr bool queries_of_listed_rows(int m, int refreshed, int d) {
  const int n = 3 * d, ksteps = d / kRouteBK;
  if (ksteps < kQuadMinSteps || m < kPartMinRows || tiles_of(m, n, kPpRows, 128) > (1 << 20)) return false;
  // (the wider tiles of all rows by their four-wave form, also where one round of them has eight waves: those are not slower)
  const GemmRoute shape = best_tile(m, n, false);
  const int t2 = tiles_of(m, n, kPpRows, 128);
  const long all = shape == GemmRoute::kPp256   ? rounds_cost(tiles_of(m, n, kPpRows, 256), 1290)
                   : shape == GemmRoute::kPp192 ? rounds_cost(tiles_of(m, n, kPpRows, 192), 1050)
                   : shape == GemmRoute::kPp128 ? rounds_cost(t2, t2 > 256 ? 848 : 800)
                                                : 0;
  const int tn = part_columns(m, n, refreshed, d);
  return rounds_cost(part_tiles(m, n, refreshed, d, tn), tn == 3 ? 1050 : 1290) + 29l * m + 37000l * 64 / ksteps < all;
}

// Row list made in the kernel: loads per wave that bring the first 256 k of an XCD's share of n weight rows into its L2, two
// rows by each of eight waves of a workgroup.  At most 8: 2 MB of the L2's 4 with a workgroup on every CU.
constexpr int ahead_loads(int n, int workgroups) {
  const int rows = workgroups / 8 * 16, loads = ((n + 7) / 8 + rows - 1) / rows;
  return loads < 8 ? loads : 8;
}

// Scored columns: whether the score is taken in the launch that projects them, rather than in one of its
// own.  Steps of four sequences that refresh a token each, one launch and two (us): k = 4096, 1024 rows 52.5 and
// 54.7, 2048 60.6 and 62.2, 2560 68.5 and 71.4, 3072 74.9 and 75.8, 4096 78.3 and 80.0, 6144 95.5 and 96.1, 8192 101.5 and
// 101.4, 12288 120.1 and 124.0, 16384 137.8 and 143.0; k = 3072, 2048 44.6 and 45.6, 2560 55.5 and 55.3, 3072 60.1 and 59.7, 4096 68.8
// and 66.4, 6144 82.4 and 83.2, 8192 82.6 and 84.9, 12288 100.6 and 105.8; k = 2048, 1024 40.6 and 42.4, 4096 54.9 and
// 54.9, 16384 91.8 and 96.7.  Up to 2048 rows and from 12288 on, where the plain projection takes larger tiles, one launch is
// the faster one; between them neither is by more than the runs differ (1 to 3 %).  The lines at k = 3072, 2560 and 8064
// rows enclose where two launches were 1 to 2 us faster with the tiles that the score's launch has now (score_proj_kernel) and
// those that the plain projection had then.
constexpr bool score_in_projection(int rows, int k) { return k < 3072 || rows <= 2560 || rows > 8064; }

// LDS of the scored-column projection once its k loop is over: bm queries, score_query_stride floats
// apart, from offset 0, and the word that says whether the workgroup is the last one
constexpr int score_query_stride(int width) { return width + 4; }
constexpr int score_arrived_offset(int bm, int width) { return bm * score_query_stride(width) * 4; }

}  // namespace dare
