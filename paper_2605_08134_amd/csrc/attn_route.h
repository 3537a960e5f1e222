// Kernel of a bf16 attention, as plain host arithmetic: no HIP here, so that the rule can be evaluated
// over its whole range without a GPU.
#pragma once

namespace dare {

enum class AttnRoute {
  kNarrow,  // blocks of 64 query rows, four key-waves; one workgroup per possible block
  kWide,    // 128 query rows, two key-waves; likewise
  kTall,    // no key split, 128 query rows (heads of 64 channels: 256); likewise
  kLaidOut, // one workgroup per CU walks blocks laid out from the refreshed-row counts
};

constexpr int kPartSteps = 8;               // least key steps (of 128) of a part where keys are cut
constexpr int kCutSteps = 2 * kPartSteps;   // key steps from which on they can be
// whether a step of up to seq tokens per sequence can use the workspace of cut keys
constexpr bool attn_may_cut(int seq) { return (seq + 127) / 128 >= kCutSteps; }

// Query rows of a sequence, at most.  many: the list holds all rows behind a frozen prefix, `active` of them (0: every row).
constexpr int attn_most_rows(int seq, bool listed, bool many, int active) {
  return listed && many && active > 0 ? active : seq;
}

// listed: the query rows are a list; many: that list holds most rows of every sequence (a frozen
// prefix), not a few (the refreshed rows); active as above.
constexpr AttnRoute attn_route(long batch, long n_heads, int seq, bool listed, bool many, bool workspace,
                               int head_dim = 128, int active = 0) {
  const long pairs = batch * n_heads;
  const int most = attn_most_rows(seq, listed, many, active);
  auto blocks = [&](int rows) { return pairs * ((most + rows - 1) / rows); };
  if (listed && !many) {
    // Refreshed rows.  Laying the blocks out on the device takes every workgroup a walk over the
    // counts, a memory latency per 64 sequences, in front of everything and again between its
    // blocks, where a key step of a block takes 0.5-1 us: it has to be short against the steps (us, first
    // with a workgroup per possible block, a few rows of each sequence refreshed: 16 x 256 tokens of 32
    // heads 31 and 21, 64 x 1024 of 8 heads 72 and 28, 8 x 2048 of 32 heads 144 and 45; the single step of a
    // short sequence it can only delay).
    const bool cut = workspace && attn_may_cut(seq);
    const AttnRoute direct = pairs < 128 ? AttnRoute::kNarrow : AttnRoute::kWide;
    const long steps = (seq + 127) / 128;
    if (batch > 8 * steps) return direct;
    if (blocks(64) >= (1l << 23)) return direct;  // (beyond the kernel's division)
    if (cut) return AttnRoute::kLaidOut;
    // Fewer than 64 pairs: narrow blocks serve them in one round unless most rows are refreshed.  No
    // more possible blocks than CUs: one round whatever is refreshed (4 x 256 of 32 heads 8.6 us, laid
    // out 9.7).
    if (pairs < 64 || blocks(direct == AttnRoute::kNarrow ? 64 : 128) <= 256) return direct;
    return AttnRoute::kLaidOut;
  }
  // Most rows of every sequence.  Heads of 128 channels: a workgroup of four waves per block and two of them on a CU,
  // unless one per CU is enough for all blocks, which then have a second wave per SIMD on the other half of the keys (us,
  // two key-waves and none, 32 heads: 1 x 1024 tokens, 256 blocks, 22.2 and 24.6; 1 x 1152 45.5 and 38.4, 1 x 1280 49.1 and 42.3, 1 x
  // 1536 57.0 and 49.2, 1 x 1920 69.2 and 62.5, 3 x 512 28.5 and 23.4, 2 x 640 31.6 and 25.6, 8 x 2048 622 and 534).  Frozen rows have no
  // block (dense steps, blocks of the whole sequence counted and of the others: 1 x 1536 tokens with 512 of them frozen 177 and 162 us,
  // 1 x 2560 of 16 heads with 768 frozen 145 and 118; heads of 64, 1 x 4096 of 16 with 2048 frozen 114 and 86).
  if (head_dim == 128) return blocks(128) > 256 ? AttnRoute::kTall : AttnRoute::kWide;
  // Heads of 64: enough rows for a block of 256 per workgroup (8 query-waves) to fill the chip: a K/V tile then feeds
  // twice the MFMAs per byte that enters LDS.
  return blocks(256) >= 256 ? AttnRoute::kTall : AttnRoute::kWide;
}

// kTall with heads of 128 channels: whether the reference exponent of the softmax moves to the second key tile's maximum, and to
// later ones with less growth.  Fewer than 256 blocks of 256 rows would be kWide's if that were as fast; its second key-wave starts
// at a maximum of its own, and one wave that keeps the first tile's is further from the exact result (130 x 129 tokens 2.12e-3
// for 1.99e-3, 1 x 1152 of 32 heads 2.30e-3 for 2.28e-3).  From 256 such blocks on kWide is no choice (4 x 512 tokens 29.5 us, kTall 24.3), and
// the move would take 0.5 us of a block (3 x 777 47.7 -> 48.3 us, 4 x 512 24.2 -> 24.5; 3 x 512, which has it, 22.6 -> 23.3).
constexpr bool attn_second_reference(long pairs, int rows) { return pairs * ((rows + 255) / 256) < 256; }

// Order of the workgroups of an XCD where there is one per possible block (kNarrow, kWide, kTall): the first blocks
// of `turn` (sequence, head)s, then their second ones, and so on; then the next `turn`.
// Listed rows, how many only the device knows: eight take turns.  One by one, a workgroup with rows lies next to
// those of the same pair without any, and an XCD, which deals its workgroups round its shader engines, keeps a
// part of its CUs idle; with all of them in one turn a pair's second block comes when its keys and values have
// left the L2 (us with one by one, 4, 8, 16, 32, all in one turn: 64 x 512 tokens of 32 heads of 128, 1 % of the rows
// 386, 129, 128, 126, 129, 130; half 495, 287, 290, 294, 298, 324; every row 530, 537, 540, 541, 526, 611;
// 64 x 256, three quarters 182, 176, 176, 176, 182, 196).
constexpr int attn_turn(int pairs, bool listed, bool many) {
  const int per_xcd = (pairs + 7) / 8;
  return listed && !many ? (per_xcd < 8 ? per_xcd : 8) : 1;
}
struct AttnPlace {
  unsigned pair, block;  // (sequence, head) of the XCD, query block
};
// (unsigned, and no division more than the case needs, none for one block per pair: this is in front of the first
// load, and a part of a block over a short sequence that shows: 128 x 64 tokens of 32 heads 82.7 -> 80.5 us)
constexpr AttnPlace attn_place(unsigned slot, unsigned per_xcd, unsigned n_blocks, unsigned turn) {
  const unsigned t = slot / (turn * n_blocks), in = slot - t * turn * n_blocks, left = per_xcd - t * turn;
  if (turn == 1) return {t, in};
  const unsigned width = left < turn ? left : turn, block = in / width;
  return {t * turn + in - block * width, block};
}

// Listed rows: workgroups per (sequence, head) that run at once, where those without rows of their own read K and V
// ahead, else 0.  They do while every block has a CU of its own and an XCD's share of K and V stays in its L2 of 4 MB.
constexpr int attn_at_once(int pairs, int seq, int head_dim) {
  const int room = (head_dim == 64 ? 512 : 256) / pairs;
  const long bytes = (long)((pairs + 7) / 8) * seq * head_dim * 4;
  return bytes <= (4l << 20) && seq > 256 && room > 1 ? room : 0;
}

// Blocks of 128 refreshed rows, per_xcd of them for the `slots` workgroups of an XCD: how many run as they are.  The rest,
// where it would leave half of the workgroups or more without one in the last round, is cut into blocks of 64 rows, of which
// that round then has at most one per workgroup (us, whole and halved: 8 x 2048 tokens of 32 heads, 6 % of them 85.3 and 78.3, 12 %
// 118.7 and 114.9; 3 x 777, half 38.4 and 35.6; 4 x 4096, 20 % 271 and 262; 6 x 1500 of 16 heads, 20 % 56.5 and 51.3).  Heads of 128
// channels only: with 64 the kernel has no register left for it.
constexpr int attn_whole_blocks(int per_xcd, int slots, bool wide) {
  const int rest = per_xcd % slots;
  return wide && 2 * rest <= slots ? per_xcd - rest : per_xcd;
}

}  // namespace dare
