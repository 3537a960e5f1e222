// Row-selected bf16 projection on the gfx950 matrix cores:
//     C[t, :] = A[t, :] . W      for t in a device-side row list
// (Alg. 1 lines 2, 6-7, 11 and Alg. 2 lines 2, 7, 11 of the paper: the Q, K, V
// and output projections, for all rows or only for the refreshed rows).
//
// Layout: A rows are k-contiguous; the weight arrives packed as Wt[n, k]
// (k-contiguous), so both MFMA operands are 16-byte runs of 8 consecutive k.
//
// A workgroup owns a BM x BN output tile and walks k in steps of 64.  Tiles of A
// and Wt go from global memory STRAIGHT INTO LDS (global_load_lds_dwordx4: lane L
// of a wave deposits its 16 bytes at wave_base + 16 L), through a ring of STAGES
// buffers, so several k-steps are in flight while the matrix cores work on the
// oldest one; no staging registers, no ds_write.  Because the LDS position is
// fixed by the lane number, bank conflicts are removed on the global side: the
// lane that owns LDS slot s of row r fetches k-chunk s ^ ((r >> 1) & 7), and the
// MFMA fragment reads apply the same XOR (measured conflict-free for 16-byte
// reads: 246 of 256 B/clk/CU).
//
// Each wave computes the TRANSPOSED tile (weight fragment as the first MFMA operand): a lane
// then owns one output row and runs of 4 consecutive output columns (8 in the large tiles),
// which gives 8- or 16-byte stores and keeps a row's values inside one lane.
//
// k-parts.  A projection with few output tiles and a long k (the scored query columns
// for all rows: 1024 x 128 x 4096) can cut k into ranges that run as separate
// workgroups; each range writes its fp32 partial products to its own slab of the fp32
// output and the consumer (the score kernel) adds the slabs in range order.  No
// atomics, no fences: the kernel boundary orders producer and consumer.
//
// Tile order.  The hardware deals workgroup ids round-robin to the 8 XCDs, each
// with its own L2.  Ids are remapped so that every XCD works on a contiguous
// range of tiles, and inside the range tiles run down groups of 8 row-tiles
// before moving to the next column-tile: the workgroups that are resident on an
// XCD at the same time then share both their A tiles and their weight tiles.
//
// Row count known only on the device (the refreshed-row list): one kernel holds
// several tile shapes and every workgroup picks the same one from the count it
// reads, so a step with 50 refreshed rows does not pay for a 256-row tile and no
// host round trip is needed.
#include <type_traits>

#include "dare_common.h"
#include "gemm_route.h"

namespace dare {
namespace {

constexpr int BK = kRouteBK;      // k per stage: one 128-byte row segment
constexpr int ROW_BYTES = BK * 2;
constexpr int GROUP_M = 8;        // row-tiles walked before the next column-tile

struct GemmDev {
  const bf16_t* a;
  const bf16_t* wt;
  const int32_t* idx;
  const int32_t* m_dev;
  bf16_t* c0;
  bf16_t* c1;
  bf16_t* c2;
  float* c32;
  int lda, n, k, m_max, ldc, seg_n, c32_cols;
  int k_parts;           // k is cut into this many ranges (1 = whole k per tile)
  long c32_part_stride;  // elements between the fp32 outputs of consecutive ranges
  const float* rope;     // rotary table, or nullptr
  int rope_cols, rope_dh, rope_seq;
  int swiglu_pairs;
  const uint8_t* sel_mask;
  int sel_batch, sel_seq;
  int32_t* sel_idx_out;
  int32_t* sel_idx_out2;
  int32_t* sel_off_out;
  int32_t* sel_count_out;
  int ahead;                // loads of weights per wave while the list is made (ahead_loads)
  // two workgroups on the halves of k of one tile (gemm_tile_pp): [tiles][2] fp32 tiles and
  // [tiles] counters; nullptr = one workgroup per tile
  float* split_tiles;
  int* split_count;
  // columns [0, part_n) for the rows of a second list only (gemm_bf16_part_kernel)
  int part_n;
  const int32_t* part_idx;
  const int32_t* part_m_dev;
};

typedef const __attribute__((address_space(1))) void* gptr_t;
typedef __attribute__((address_space(3))) void* lptr_t;
typedef const __attribute__((address_space(3))) int32_t* lds_idx_t;  // a row list held in LDS

// Token ids of listed rows: from the list in LDS when the kernel derived it itself, else from the
// caller's list, else the rows themselves.  (One branch around all of them: a branch per row takes
// longer than the reads.)
template <int N>
__device__ __forceinline__ void row_tokens(const int32_t* __restrict__ gidx, lds_idx_t lidx, const int (&row)[N],
                                           int (&tok)[N]) {
  if (lidx) {
#pragma unroll
    for (int i = 0; i < N; ++i) tok[i] = lidx[row[i]];
  } else if (gidx) {
#pragma unroll
    for (int i = 0; i < N; ++i) tok[i] = gidx[row[i]];
  } else {
#pragma unroll
    for (int i = 0; i < N; ++i) tok[i] = row[i];
  }
}

// Wait until at most N of this wave's vector-memory operations are outstanding
// and all of its LDS reads have returned, then join the workgroup barrier.
// Written as one asm statement with a memory clobber: __syncthreads() would add a
// release fence, and the compiler answers a fence with vmcnt(0), which would
// drain the whole ring of in-flight k-steps.
template <int N>
__device__ __forceinline__ void wait_vmcnt_and_barrier() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// The same where `ahead` (0 .. MAX, or more for MAX; the same in all waves) stages of LOADS each may be outstanding
template <int LOADS, int MAX>
__device__ __forceinline__ void wait_stages_and_barrier(const int ahead) {
  if constexpr (MAX > 0) {
    if (ahead < MAX) return wait_stages_and_barrier<LOADS, MAX - 1>(ahead);
  }
  wait_vmcnt_and_barrier<LOADS * MAX>();
}

template <int BM, int BN, int STAGES>
constexpr int smem_bytes() {
  return STAGES * (BM + BN) * ROW_BYTES;
}

// silu(g) = g / (1 + exp(-g)), by hand: reciprocal, product, one correction, special values by v_div_fixup.  Over all 2^32 values of g
// it has the bits of the compiler's division, which does not know that the divisor is 1 or more and takes twice as long.
// SCALED: divisors above 2^126 (g below -87.336), whose reciprocal is flushed to 0, are multiplied by a power of two; without it only
// for g of kGateLow or more.
constexpr float kGateLow = -87.0f;
template <bool SCALED = true>
__device__ __forceinline__ float silu(float g) {
  const float scale = SCALED && g < kGateLow ? 0x1p-32f : 1.0f;
  const float d = fmaf(__expf(-g), scale, scale), r = __builtin_amdgcn_rcpf(d), q = g * r;
  return __builtin_amdgcn_div_fixupf(fmaf(fmaf(-d, q, g), r, q) * scale, d, g);
}

// Epilogue of a wave tile: W (4 or 8) neighbouring output columns col[j] .. col[j] + W - 1 (col[j] a multiple
// of W; a segment, whose width is a multiple of 32, holds all of them) of tokens tok[i], live[i] or not,
// value(i, j, e) each.  Plain: the fp32 copy of the scored columns (before any rotation), then
// rotation, rounding and the store into the column's segment.  Gated: (gate, up) pairs, W / 2 outputs
// silu(gate) * up from column col / 2 on.
// What a launch asks for is settled outside the loops and what a column needs outside that over the rows: decided
// at every store, with the kernel's arguments read again and a division each for segment and
// position, the epilogue was as long as a third of the k loop (its gain is part of gemm_tile16's figures).
template <int W, int TM, int TN, class Value>
__device__ __forceinline__ void store_tile(const GemmDev& p, float* c32, const int (&tok)[TM], const bool (&live)[TM],
                                           const int (&col)[TN], Value value) {
  static_assert(W == 4 || W == 8, "columns of a store");
  typedef __bf16 out_t __attribute__((ext_vector_type(W)));
  typedef __bf16 half_t __attribute__((ext_vector_type(W / 2)));
  if (p.swiglu_pairs) {
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      bf16_t* row = p.c0 + (long)tok[i] * p.ldc;
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        half_t o;
#pragma unroll
        for (int e = 0; e < W / 2; ++e) {
          const float g = value(i, j, 2 * e);
          o[e] = (bf16_t)(silu(g) * value(i, j, 2 * e + 1));
        }
        if (live[i] && col[j] < p.n) *reinterpret_cast<half_t*>(row + (col[j] >> 1)) = o;
      }
    }
    return;
  }
  int pos[TM];
  if (p.rope) {
#pragma unroll
    for (int i = 0; i < TM; ++i) pos[i] = (unsigned)tok[i] % (unsigned)p.rope_seq;
  }
  const long ldc = p.ldc;
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int c = col[j];
    if (c >= p.n) continue;
    float v[TM][W];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int e = 0; e < W; ++e) v[i][e] = value(i, j, e);
    if (c32) {
#pragma unroll
      for (int h = 0; h < W; h += 4)
        if (c + h < p.c32_cols) {
#pragma unroll
          for (int i = 0; i < TM; ++i)
            if (live[i])
              *reinterpret_cast<f32x4*>(c32 + (long)tok[i] * p.c32_cols + c + h) =
                  f32x4{v[i][h], v[i][h + 1], v[i][h + 2], v[i][h + 3]};
        }
    }
    const int seg = (c >= p.seg_n) + (c >= 2 * p.seg_n);
    bf16_t* cbase = seg == 0 ? p.c0 : (seg == 1 ? p.c1 : p.c2);
    if (!cbase) continue;
    cbase += c - seg * p.seg_n;
    if (p.rope) {
#pragma unroll
      for (int h = 0; h < W; h += 4)
        if (c + h < p.rope_cols) {
          const float* table = p.rope + (((unsigned)(c + h) % (unsigned)p.rope_dh) >> 1) * 2;
          f32x4 cs[TM];
#pragma unroll
          for (int i = 0; i < TM; ++i) cs[i] = *reinterpret_cast<const f32x4*>(table + (long)pos[i] * p.rope_dh);
#pragma unroll
          for (int i = 0; i < TM; ++i) rope_rotate4(cs[i], v[i][h], v[i][h + 1], v[i][h + 2], v[i][h + 3]);
        }
    }
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      out_t o;
#pragma unroll
      for (int e = 0; e < W; ++e) o[e] = (bf16_t)v[i][e];
      if (live[i]) *reinterpret_cast<out_t*>(cbase + tok[i] * ldc) = o;
    }
  }
}

// Tile order: GROUP_M row-tiles per column step (the tiles that run at the same time on one
// XCD then share few distinct A and W tiles).
__device__ __forceinline__ void tile_of_unit(const int unit, const int tiles_m, const int tiles_n, int& tile_m,
                                             int& tile_n) {
  const int group_size = GROUP_M * tiles_n;
  const int first_m = (unit / group_size) * GROUP_M;
  const int rows_in_group = tiles_m - first_m < GROUP_M ? tiles_m - first_m : GROUP_M;
  const int rem = unit % group_size;
  tile_m = first_m + rem % rows_in_group;
  tile_n = rem / rows_in_group;
}

// A range of the k (one of k_parts) of an output tile of C for m rows, computed by the WAVES_M * WAVES_N waves of a
// workgroup in smem_bytes<BM, BN, STAGES>() bytes of LDS.
template <int BM, int BN, int WAVES_M, int WAVES_N, int STAGES>
__device__ __forceinline__ void gemm_tile(const GemmDev& p, const int m, unsigned char* smem) {
  constexpr int NW = WAVES_M * WAVES_N;
  constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;
  constexpr int TM = WM / 32, TN = WN / 32;
  constexpr int STAGE_BYTES = (BM + BN) * ROW_BYTES;
  constexpr int GROUPS = (BM + BN) / 8;  // 8-row groups = one wave load each
  constexpr int LPW = GROUPS / NW;       // loads per wave per stage
  static_assert(WM % 32 == 0 && WN % 32 == 0, "wave tile must be a multiple of 32 x 32");
  static_assert(GROUPS % NW == 0, "row groups must divide among the waves");
  static_assert(LPW * (STAGES - 1) < 64, "vmcnt range");

  // ---- which tile: XCD-contiguous ranges, GROUP_M row-tiles per column step ----
  // (the k-ranges of one tile are neighbours in this order)
  const int parts = p.k_parts;
  const int tiles_m = (m + BM - 1) / BM, tiles_n = (p.n + BN - 1) / BN;
  const int total = tiles_m * tiles_n * parts;
  const int per_xcd = (total + 7) >> 3;
  const int slot = blockIdx.x >> 3;
  if (slot >= per_xcd) return;
  const int unit = (blockIdx.x & 7) * per_xcd + slot;
  if (unit >= total) return;
  const int logical = unit / parts, part = unit - logical * parts;
  int tile_m, tile_n;
  tile_of_unit(logical, tiles_m, tiles_n, tile_m, tile_n);
  const int m0 = tile_m * BM, n0 = tile_n * BN;

  // (the wave number as a scalar: LDS addresses of the global -> LDS loads go through M0, and a
  // wave number held in a vector register would send every one of them through v_readfirstlane)
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wave_m = wave % WAVES_M, wave_n = wave / WAVES_M;
  const int l32 = lane & 31, half = lane >> 5;

  // this workgroup's k-range, in k-steps (the host makes parts divide the step count)
  const int KT = p.k / BK / parts;
  const int kt0 = part * KT;

  // ---- global -> LDS assignment: wave w issues loads for row groups w*LPW .. +LPW
  // (rows 0..BM-1 are A rows, BM..BM+BN-1 are weight rows).  Lane L of a load owns
  // row (L >> 3) of the group and LDS slot (L & 7); it fetches the k-chunk that
  // the swizzle puts into that slot.  Rows past the end re-read the last row.
  const bf16_t* src[LPW];
  int row_in[LPW], tok_in[LPW];
#pragma unroll
  for (int i = 0; i < LPW; ++i) {
    const int row = m0 + (wave * LPW + i) * 8 + (lane >> 3);
    row_in[i] = row < m ? row : m - 1;
  }
  row_tokens(p.idx, nullptr, row_in, tok_in);
#pragma unroll
  for (int i = 0; i < LPW; ++i) {
    const int r = (wave * LPW + i) * 8 + (lane >> 3);  // row within the stage
    const int chunk = (lane & 7) ^ ((r >> 1) & 7);
    if (r < BM) {
      src[i] = p.a + (long)tok_in[i] * p.lda + chunk * 8 + kt0 * BK;
    } else {
      int col = n0 + (r - BM);
      col = col < p.n ? col : p.n - 1;
      src[i] = p.wt + (long)col * p.k + chunk * 8 + kt0 * BK;
    }
  }
  int row_out[TM], tok_out[TM];
  bool live_out[TM];
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int row = m0 + wave_m * WM + i * 32 + l32;
    live_out[i] = row < m;
    row_out[i] = row < m ? row : m - 1;
  }
  row_tokens(p.idx, nullptr, row_out, tok_out);
  auto issue_loads = [&](int kt, int buf) __attribute__((always_inline)) {
    unsigned char* base = smem + buf * STAGE_BYTES + wave * LPW * 8 * ROW_BYTES;
#pragma unroll
    for (int i = 0; i < LPW; ++i)
      __builtin_amdgcn_global_load_lds((gptr_t)(src[i] + kt * BK),
                                       (lptr_t)(base + i * 8 * ROW_BYTES), 16, 0, 0);
  };

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  // fragment read offsets: row (wave tile base + 32 i + l32), k-chunk 2 ks + half,
  // stored at slot chunk ^ ((row >> 1) & 7); the tile bases are multiples of 32,
  // so the XOR term depends on l32 only
  constexpr int KS = BK / 16;
  const int sw = (l32 >> 1) & 7;
  int koff[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) koff[ks] = ((ks * 2 + half) ^ sw) * 16;
  const int a_row_off = (wave_m * WM + l32) * ROW_BYTES;
  const int b_row_off = (BM + wave_n * WN + l32) * ROW_BYTES;

  // ---- pipeline: STAGES-1 k-steps in flight ahead of the one being multiplied.
  // Loads of k-steps past the end are issued on the last valid k-step again (into
  // a buffer nobody reads any more), so the count of outstanding loads per wave is
  // the same in every iteration and one vmcnt value serves the whole loop.
  //
  // MFMA operands are double-buffered in registers: all fragments of k-step kt+1 are fetched
  // after the first PRE MFMAs of k-step kt and arrive under the rest.  The barrier that publishes
  // k-step kt+1 sits right before that fetch: by then every LDS read of k-step kt has been issued
  // and (lgkmcnt 0) has completed, so its buffer may be refilled after the barrier.
  // The scheduling fences keep the compiler from sinking the LDS reads back down
  // to their first use, which would undo the register double buffering.
  bf16x8 fa[2][KS][TM], fb[2][KS][TN];
  auto load_frags = [&](int buf, int set) __attribute__((always_inline)) {
    const unsigned char* st = smem + buf * STAGE_BYTES;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
        fa[set][ks][i] = *reinterpret_cast<const bf16x8*>(st + a_row_off + i * 32 * ROW_BYTES + koff[ks]);
#pragma unroll
      for (int j = 0; j < TN; ++j)
        fb[set][ks][j] = *reinterpret_cast<const bf16x8*>(st + b_row_off + j * 32 * ROW_BYTES + koff[ks]);
    }
  };
  // MFMAs [first, last) of the KS x TM x TN grid of one fragment set
  constexpr int NMMA = KS * TM * TN;
  constexpr int PRE = NMMA >= 8 ? 2 : 1;
  auto mma = [&](int set, int first, int last) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < NMMA; ++t) {
      if (t < first || t >= last) continue;
      const int ks = t / (TM * TN), i = (t / TN) % TM, j = t % TN;
      acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[set][ks][j], fa[set][ks][i], acc[i][j], 0, 0, 0);
    }
  };

#pragma unroll
  for (int s = 0; s < STAGES - 1; ++s) issue_loads(s < KT ? s : KT - 1, s);
  wait_vmcnt_and_barrier<LPW*(STAGES - 2)>();
  load_frags(0, 0);
  // two k-steps per trip so that the fragment set index is a compile-time constant
  // (a run-time index would push the fragment arrays out of registers)
  auto kstep = [&](int kt, auto set_c) __attribute__((always_inline)) {
    constexpr int SET = decltype(set_c)::value;
    const int nxt = kt + STAGES - 1;
    issue_loads(nxt < KT ? nxt : KT - 1, nxt % STAGES);
    mma(SET, 0, PRE);
    __builtin_amdgcn_sched_barrier(0);
    wait_vmcnt_and_barrier<LPW*(STAGES - 2)>();
    load_frags((kt + 1) % STAGES, SET ^ 1);
    __builtin_amdgcn_sched_barrier(0);
    mma(SET, PRE, NMMA);
    __builtin_amdgcn_sched_barrier(0);
  };
  int kt = 0;
  for (; kt + 1 < KT; kt += 2) {
    kstep(kt, std::integral_constant<int, 0>{});
    kstep(kt + 1, std::integral_constant<int, 1>{});
  }
  if (kt < KT) kstep(kt, std::integral_constant<int, 0>{});
  wait_vmcnt<0>();

  float* c32 = p.c32 + part * p.c32_part_stride;
  // Epilogue.  acc[i][j][r] = C[row, col] with
  //   row = m0 + wave_m*WM + i*32 + l32
  //   col = n0 + wave_n*WN + j*32 + (r/4)*8 + half*4 + r%4
  int col[4 * TN];
#pragma unroll
  for (int j = 0; j < 4 * TN; ++j) col[j] = n0 + wave_n * WN + j * 8 + half * 4;
  store_tile<4>(p, c32, tok_out, live_out, col,
                [&](int i, int j, int e) __attribute__((always_inline)) { return acc[i][j >> 2][(j & 3) * 4 + e]; });
}

// Tiles that the CUs get one of, or few: eight waves, v_mfma_f32_16x16x32_bf16 (wave tiles in units of
// 16, so that eight waves can share a 128 x 96 tile: 129-256 refreshed rows of a 12288-wide output then
// make 256 workgroups of 8 waves, where the 32-wide shape allows 192 workgroups of 128 x 128).  LDS
// layout as in gemm_tile; a fragment is 16 rows x 32 k (lane L: row L & 15, k-chunk L >> 4), a k-step
// holds two such slices, and all fragments of the next k-step are fetched under the MFMAs of the
// current one.  vblock is the workgroup's (virtual) block id: one that walks several tiles calls this
// once per pass with block id + pass * grid size; the result says whether that id held a tile.
// What bounds it is the pull of a CU: the operands come at most at 64 B per cycle, at 100 GB/s where
// lines come from beyond the L2 (1024 x 4096 x 4096: loads alone 26 us of 33, MFMAs alone 20).  So the whole ring is
// kept in flight (the stage of k-step kt is filled again for kt + STAGES as soon as the barrier says that its
// fragments are in registers) and the loads of a k-step are issued one by one between its MFMAs: in a
// row, a wave that waits for a place in the queue keeps its MFMAs waiting as well.  us, before (STAGES - 1
// stages in flight, loads in a row, 32-wide MFMAs for 128 x 128, the epilogue before store_tile) and now, weights in the
// last-level cache: all rows, 1024 x 4096 x 4096 41.3 and 36.3, 512 x 8192 41.5 and 35.3; listed rows, 205 x 12288 32.2 and
// 31.4 (weights from HBM 39.4 and 37.6), 205 x 4096 16.7 and 16.4, 512 x 8192 43.3 and 37.1, but 100 x 12288 (128 x 48) 23.1
// and 23.8.  (The order of a sum over k is that of the instruction: 128 x 128 tiles sum 32 products at a time where they
// summed 16, results differ from then by single bf16 roundings.)  The k of a k-step halved
// between two groups of four waves with twice the wave tile (half the fragment reads) is no faster.
// Some waves repeat the last group of rows (128 x 96: 32 loads for 28 groups).
template <int BM, int BN, int WAVES_M, int WAVES_N, int STAGES>
__device__ __forceinline__ bool gemm_tile16(const GemmDev& p, const int m, unsigned char* smem, const int tid,
                                            const int vblock, lds_idx_t lidx = nullptr,
                                            const int forced_tile_m = -1, const int forced_tile_n = 0) {
  constexpr int NW = WAVES_M * WAVES_N;
  constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;
  constexpr int TM = WM / 16, TN = WN / 16;
  constexpr int STAGE_BYTES = (BM + BN) * ROW_BYTES;
  constexpr int GROUPS = (BM + BN) / 8;
  constexpr int LPW = (GROUPS + NW - 1) / NW;  // surplus loads repeat the last group
  constexpr int KS = BK / 32;
  static_assert(WM % 16 == 0 && WN % 16 == 0, "wave tile must be a multiple of 16 x 16");
  static_assert(STAGES >= 3 && LPW * (STAGES - 1) < 64, "vmcnt range");

  const int tiles_m = (m + BM - 1) / BM, tiles_n = (p.n + BN - 1) / BN;
  int tile_m, tile_n;
  if (forced_tile_m >= 0) {  // the caller names the tile
    tile_m = forced_tile_m;
    tile_n = forced_tile_n;
  } else {
    const int total = tiles_m * tiles_n;
    const int per_xcd = (total + 7) >> 3;
    const int slot = vblock >> 3;
    if (slot >= per_xcd) return false;
    const int unit = (vblock & 7) * per_xcd + slot;
    if (unit >= total) return false;
    tile_of_unit(unit, tiles_m, tiles_n, tile_m, tile_n);
  }
  const int m0 = tile_m * BM, n0 = tile_n * BN;

  // (the wave number as a scalar: LDS addresses of the global -> LDS loads go through M0, and a
  // wave number held in a vector register would send every one of them through v_readfirstlane)
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wave_m = wave % WAVES_M, wave_n = wave / WAVES_M;
  const int l16 = lane & 15, kq = lane >> 4;
  const int KT = p.k / BK;

  const bf16_t* src[LPW];
  int grp[LPW], row_in[LPW], tok_in[LPW];
#pragma unroll
  for (int i = 0; i < LPW; ++i) {
    grp[i] = wave * LPW + i < GROUPS ? wave * LPW + i : GROUPS - 1;
    const int row = m0 + grp[i] * 8 + (lane >> 3);
    row_in[i] = row < m ? row : m - 1;
  }
  row_tokens(p.idx, lidx, row_in, tok_in);
#pragma unroll
  for (int i = 0; i < LPW; ++i) {
    const int r = grp[i] * 8 + (lane >> 3);
    const int chunk = (lane & 7) ^ ((r >> 1) & 7);
    if (r < BM) {
      src[i] = p.a + (long)tok_in[i] * p.lda + chunk * 8;
    } else {
      int col = n0 + (r - BM);
      col = col < p.n ? col : p.n - 1;
      src[i] = p.wt + (long)col * p.k + chunk * 8;
    }
  }
  int row_out[TM], tok_out[TM];
  bool live_out[TM];
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int row = m0 + wave_m * WM + i * 16 + l16;
    live_out[i] = row < m;
    row_out[i] = row < m ? row : m - 1;
  }
  row_tokens(p.idx, lidx, row_out, tok_out);
  // TRIM: nothing is loaded past the last k-step (steps of 1 x 1024 x 4096, half of the tokens refreshed: 155.5 ->
  // 154.2 us).  Otherwise the loads of k-steps past the end repeat the last one, into a stage that nobody reads any
  // more, so that one loop with one wait serves all k-steps: the last ones of a small tile take less than
  // fetching code of their own does (2 x 201 x 512 28.4 us as it is and 29.6 with TRIM, 4 of 1024 rows 61.0 and 62.5).
  constexpr bool TRIM = TM * TN >= 6;
  auto issue_load = [&](int i, int kt) __attribute__((always_inline)) {
    const int k = TRIM || kt < KT ? kt : KT - 1;
    __builtin_amdgcn_global_load_lds((gptr_t)(src[i] + k * BK),
                                     (lptr_t)(smem + (kt % STAGES) * STAGE_BYTES + grp[i] * 8 * ROW_BYTES), 16, 0, 0);
  };

  f32x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  // fragment offsets: row (base + 16 i + l16), chunk 4 ks + kq at slot chunk ^ ((row >> 1) & 7); the
  // bases are multiples of 16, so the XOR term depends on l16 only
  const int sw = (l16 >> 1) & 7;
  int koff[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) koff[ks] = ((ks * 4 + kq) ^ sw) * 16;
  const int a_row_off = (wave_m * WM + l16) * ROW_BYTES;
  const int b_row_off = (BM + wave_n * WN + l16) * ROW_BYTES;

  bf16x8 fa[2][KS][TM], fb[2][KS][TN];
  auto load_frags = [&](int kt, int set) __attribute__((always_inline)) {
    const unsigned char* st = smem + (kt % STAGES) * STAGE_BYTES;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
        fa[set][ks][i] = *reinterpret_cast<const bf16x8*>(st + a_row_off + i * 16 * ROW_BYTES + koff[ks]);
#pragma unroll
      for (int j = 0; j < TN; ++j)
        fb[set][ks][j] = *reinterpret_cast<const bf16x8*>(st + b_row_off + j * 16 * ROW_BYTES + koff[ks]);
    }
  };
  constexpr int NMMA = KS * TM * TN, PRE = NMMA / 4 > 0 ? NMMA / 4 : 1;
  auto mma = [&](int set, int first, int last) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < NMMA; ++t) {
      if (t < first || t >= last) continue;
      const int ks = t / (TM * TN), i = (t / TN) % TM, j = t % TN;
      acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[set][ks][j], fa[set][ks][i], acc[i][j], 0, 0, 0);
    }
  };

#pragma unroll
  for (int s = 0; s < STAGES; ++s)
    if (!TRIM || s < KT) {
#pragma unroll
      for (int i = 0; i < LPW; ++i) issue_load(i, s);
    }
  wait_stages_and_barrier<LPW, STAGES - 1>(TRIM ? KT - 1 : STAGES - 1);
  load_frags(0, 0);
  // k-step kt: the barrier publishes stage kt + 1 and, as every wave's fragments of kt have arrived, frees
  // the stage of kt.  (Two k-steps per trip so that the fragment set index is a compile-time constant.)
  // END: one of the last k-steps, which has nothing left to load and waits for as many loads as are under way.
  auto kstep = [&](int kt, auto set_c, auto end_c) __attribute__((always_inline)) {
    constexpr int SET = decltype(set_c)::value;
    constexpr bool END = decltype(end_c)::value;
    mma(SET, 0, PRE);
    __builtin_amdgcn_sched_barrier(0);
    if (!END || kt + 1 < KT) {
      if constexpr (END)
        wait_stages_and_barrier<LPW, STAGES - 2>(KT - 2 - kt);
      else
        wait_vmcnt_and_barrier<LPW*(STAGES - 2)>();
      __builtin_amdgcn_sched_barrier(0);
      load_frags(kt + 1, SET ^ 1);
    }
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (END) {
      mma(SET, PRE, NMMA);
    } else {
#pragma unroll
      for (int i = 0; i < LPW; ++i) {
        mma(SET, PRE + (NMMA - PRE) * i / LPW, PRE + (NMMA - PRE) * (i + 1) / LPW);
        __builtin_amdgcn_sched_barrier(0);
        issue_load(i, kt + STAGES);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
  using Yes = std::true_type;
  using No = std::false_type;
  using Set0 = std::integral_constant<int, 0>;
  using Set1 = std::integral_constant<int, 1>;
  int kt = 0;
  const int loading = TRIM ? KT - STAGES : KT;
  for (; kt + 1 < loading; kt += 2) {
    kstep(kt, Set0{}, No{});
    kstep(kt + 1, Set1{}, No{});
  }
  if constexpr (!TRIM) {
    if (kt < KT) kstep(kt, Set0{}, No{});
    kt = KT;
  } else if (kt < loading) {  // an odd number of k-steps load: the last ones begin with set 1
    kstep(kt, Set0{}, No{});
    kstep(++kt, Set1{}, Yes{});
    ++kt;
  }
  for (; kt < KT; kt += 2) {
    kstep(kt, Set0{}, Yes{});
    if (kt + 1 < KT) kstep(kt + 1, Set1{}, Yes{});
  }
  wait_vmcnt<0>();

  // acc[i][j][e] = C[row, col]: row = m0 + wave_m*WM + 16 i + l16, col = n0 + wave_n*WN + 16 j + 4 kq + e
  int col[TN];
#pragma unroll
  for (int j = 0; j < TN; ++j) col[j] = n0 + wave_n * WN + j * 16 + kq * 4;
  store_tile<4>(p, p.c32, tok_out, live_out, col,
                [&](int i, int j, int e) __attribute__((always_inline)) { return acc[i][j][e]; });
  return true;
}

// ---- large tiles: 256 x (64 TN), eight waves in two groups that take turns ----------------
// (listed rows; all rows in 256 x 128, with k cut too, and in one round of the wider ones)
// Waves w and w + 4 sit on the same SIMD.  Waves 0-3 (group 0) own the left half of the tile's
// columns, waves 4-7 (group 1) the right half, each wave 64 rows x 32 TN columns.  A k-step of 64 is
// cut into TN phases, one per block of 32 columns, and a phase into a memory part (fragment
// reads of the phase from LDS, waits) and a matrix part (16 MFMAs), with a workgroup barrier
// after each.  Group 1 runs one barrier behind group 0, so on every SIMD one wave multiplies while
// the other reads: neither the LDS reads nor the barriers leave the matrix pipe idle.
//   * The global -> LDS loads are issued between the MFMAs of the matrix part, one or two per phase
//     and wave.  In the memory part, or ahead of its reads, the vector-memory queue holds up the
//     wave that the others wait for: 2930 and 3870 cycles per k-step of a 256 x 256 tile, against
//     2300 between the MFMAs (2048 is what the MFMAs alone take).
//   * v_mfma_f32_16x16x32_bf16 and not 32x32x16: it moves fewer accumulator registers per flop, and
//     these kernels run at the power limit (1.6-1.9 GHz of 2.4 under load): 16384 x 12288 x 4096 takes
//     1140 us against 1285 us although a k-step has 9 % more cycles.
//   * The weight rows of a fragment are permuted (row 8 a + b of a 32-row block feeds result row
//     4 a + b of the first MFMA, row 8 a + 4 + b the second, a, b = 0 .. 3), so that a lane ends up with
//     eight neighbouring output columns: 16-byte stores, half the store requests (the epilogue of a
//     256 x 256 tile: 5.1 against 11 thousand cycles).  The chunk XOR of a weight row follows that
//     order ((row >> 1) & 1 | ((row >> 3) & 3) << 1), which keeps the reads conflict-free.
//   * LDS: two stages (three for TN = 2), each freed region by region.  The A rows of k-step kt are read in phase 0 only
//     and column block j in phase j (block 0 already in the last phase of kt - 1); a region is filled
//     again for kt + 2 from the phase after on, so a load has 3.5 (TN = 3) or 4.5 phases (TN = 4) of
//     512 MFMA cycles to arrive.
// Measured with gathered-row support and all (us, before: one k-loop that every wave runs in step):
// 16384 x 12288 x 4096 1540 -> 1140 (1.45 PFLOP/s), 1024 x 12288 x 4096 98 -> 78, 1024 x 24576 x 4096
// 206 -> 154.  TN = 2 against 128 x 128 tiles: 2048 x 4096 x 4096 83 -> 59; with the k of a tile cut over
// two workgroups (below; 64 to 128 tiles, which leave half of the CUs idle, and a long k), inside a
// model step: 1024 x 4096 x 12288 122 -> 97.  A k-step takes 1610 cycles for 1024 of MFMAs:
// every byte of LDS written or read for it at 128 B per cycle is 1400.
// The last k-steps load nothing and wait for what is under way: a launch of one round had two k-steps of 64
// pulled in vain and the last load's latency at its end.  Steps: 3 x 777, outputs reused 285.7 -> 282.1 us, 8 x 2048
// refreshed 534.8 -> 525.2, dense block 2323 -> 2300; a dense step of 1024 tokens 148.6 -> 148.9.
template <int TN>
constexpr int pp_stages() { return TN == 2 ? 3 : 2; }
template <int TN>
constexpr int pp_smem_bytes() {
  return pp_stages<TN>() * (kPpRows + 64 * TN) * ROW_BYTES;
}
// chunk XOR of row r of a 32-row weight block
__device__ __forceinline__ int pp_bkey(int r) { return ((r >> 1) & 1) | (((r >> 3) & 3) << 1); }

// vblock, lidx and the result as in gemm_tile16; called by all 512 threads.
template <int TN, bool SPLIT = false>
__device__ __forceinline__ bool gemm_tile_pp(const GemmDev& p, const int m, unsigned char* smem, const int vblock,
                                             lds_idx_t lidx = nullptr) {
  static_assert(TN >= 2 && TN <= 4, "column blocks of 32 per wave");
  static_assert(!SPLIT || TN == 2, "k is cut for the narrow tile only");
  constexpr int BM = kPpRows, BN = 64 * TN;
  constexpr int ASZ = BM * ROW_BYTES, BSZ = BN * ROW_BYTES, STAGE_BYTES = ASZ + BSZ, STAGES = pp_stages<TN>();
  constexpr int PARTS = SPLIT ? 2 : 1;

  const int tiles_m = (m + BM - 1) / BM, tiles_n = (p.n + BN - 1) / BN;
  const int total = tiles_m * tiles_n * PARTS;
  const int per_xcd = (total + 7) >> 3;
  const int slot = vblock >> 3;
  if (slot >= per_xcd) return false;
  const int unit = (vblock & 7) * per_xcd + slot;
  if (unit >= total) return false;
  const int tile = unit / PARTS;
  int tile_m, tile_n;
  tile_of_unit(tile, tiles_m, tiles_n, tile_m, tile_n);
  const int m0 = tile_m * BM, n0 = tile_n * BN;

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int grp = wave >> 2, wm = wave & 3;
  const int l16 = lane & 15, kq = lane >> 4;
  const int KT = p.k / BK / PARTS;
  const int k_first = SPLIT ? (unit & 1) * KT * BK : 0;

  // ---- global -> LDS: per k-step a wave loads 4 groups of 8 A rows and one group of 8 weight rows
  // of each column block (block j: rows 32 j .. of the left and of the right half, 64 in all).
  // Rows past the end re-read the last one.
  const bf16_t* src_a[4];
  const bf16_t* src_b[TN];
  int row_in[4], tok_in[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int row = m0 + (wave * 4 + i) * 8 + (lane >> 3);
    row_in[i] = row < m ? row : m - 1;
  }
  row_tokens(p.idx, lidx, row_in, tok_in);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = (wave * 4 + i) * 8 + (lane >> 3);
    src_a[i] = p.a + (long)tok_in[i] * p.lda + ((lane & 7) ^ ((r >> 1) & 7)) * 8 + k_first;
  }
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int r = wave * 8 + (lane >> 3);
    int col = n0 + (r >> 5) * (32 * TN) + j * 32 + (r & 31);
    col = col < p.n ? col : p.n - 1;
    src_b[j] = p.wt + (long)col * p.k + ((lane & 7) ^ pp_bkey(r & 31)) * 8 + k_first;
  }
  int row_out[4], tok_out[4];
  bool live_out[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int row = m0 + wm * 64 + i * 16 + l16;
    live_out[i] = row < m;
    row_out[i] = row < m ? row : m - 1;
  }
  row_tokens(p.idx, lidx, row_out, tok_out);
  // (in front of the loop, k-steps past the end of a short k re-read the last one into a region that nobody
  // reads, so that the loads in flight are at least those that the loop counts; the loop loads nothing past the end)
  auto stage = [&](int kt) __attribute__((always_inline)) { return smem + (kt % STAGES) * STAGE_BYTES; };
  auto load_a = [&](int i, int kt, int k) __attribute__((always_inline)) {
    __builtin_amdgcn_global_load_lds((gptr_t)(src_a[i] + k * BK), (lptr_t)(stage(kt) + (wave * 4 + i) * 1024), 16, 0, 0);
  };
  auto load_b = [&](int j, int kt, int k) __attribute__((always_inline)) {
    __builtin_amdgcn_global_load_lds((gptr_t)(src_b[j] + k * BK),
                                     (lptr_t)(stage(kt) + ASZ + j * 64 * ROW_BYTES + wave * 1024), 16, 0, 0);
  };

  f32x4 acc[4][2 * TN];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 2 * TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  const int a_off = (wm * 64 + l16) * ROW_BYTES;
  int a_koff[2], b_koff[2][2];
  const int brow = (l16 >> 2) * 8 + (l16 & 3);
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) {
    a_koff[ks] = ((ks * 4 + kq) ^ ((l16 >> 1) & 7)) * 16;
#pragma unroll
    for (int h = 0; h < 2; ++h)
      b_koff[h][ks] = (grp * 32 + brow + 4 * h) * ROW_BYTES + (((ks * 4 + kq) ^ pp_bkey(brow + 4 * h)) * 16);
  }
  bf16x8 fa[4][2], fb[2][2][2];  // A fragments of a k-step; weight fragments of two column blocks
  auto read_a = [&](int kt) __attribute__((always_inline)) {
    const unsigned char* st = stage(kt) + a_off;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int i = 0; i < 4; ++i) fa[i][ks] = *reinterpret_cast<const bf16x8*>(st + i * 16 * ROW_BYTES + a_koff[ks]);
  };
  auto read_b = [&](int set, int j, int kt) __attribute__((always_inline)) {
    const unsigned char* st = stage(kt) + ASZ + j * 64 * ROW_BYTES;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int h = 0; h < 2; ++h) fb[set][h][ks] = *reinterpret_cast<const bf16x8*>(st + b_koff[h][ks]);
  };
  // MFMAs [first, last) of the 16 of column block j
  auto mma = [&](int set, int j, int first, int last) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < 16; ++t) {
      if (t < first || t >= last) continue;
      const int ks = t >> 3, i = (t >> 1) & 3, h = t & 1;
      acc[i][j * 2 + h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[set][h][ks], fa[i][ks], acc[i][j * 2 + h], 0, 0, 0);
    }
  };
  // end of a memory part: all but N of the wave's loads have landed, its LDS reads have returned
  auto end_mem = [&](auto n_c) __attribute__((always_inline)) {
    __builtin_amdgcn_sched_barrier(0);
    wait_vmcnt_and_barrier<decltype(n_c)::value>();
    __builtin_amdgcn_sched_barrier(0);
  };
  // a matrix part: the MFMAs of column block j with up to four loads between them
  auto matrix = [&](int set, int j, auto l1, auto l2, auto l3, auto l4) __attribute__((always_inline)) {
    __builtin_amdgcn_s_setprio(1);
    mma(set, j, 0, 4);
    __builtin_amdgcn_sched_barrier(0);
    l1();
    __builtin_amdgcn_sched_barrier(0);
    mma(set, j, 4, 8);
    __builtin_amdgcn_sched_barrier(0);
    l2();
    __builtin_amdgcn_sched_barrier(0);
    mma(set, j, 8, 12);
    __builtin_amdgcn_sched_barrier(0);
    l3();
    __builtin_amdgcn_sched_barrier(0);
    mma(set, j, 12, 14);
    __builtin_amdgcn_sched_barrier(0);
    l4();
    __builtin_amdgcn_sched_barrier(0);
    mma(set, j, 14, 16);
    __builtin_amdgcn_s_setprio(0);
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  auto none = []() __attribute__((always_inline)) {};
#define DARE_N(n) std::integral_constant<int, n>{}
#define DARE_A(on, i, d) [&]() __attribute__((always_inline)) { if constexpr (on) load_a(i, kt + d, kt + d); }
#define DARE_B(on, j, d) [&]() __attribute__((always_inline)) { if constexpr (on) load_b(j, kt + d, kt + d); }

  // Loads in the order in which they are needed: block 0 of a k-step, its A rows, its blocks
  // 1 .. TN - 1.  The counts below are the loads issued after the last one that the next phase reads.
  const int k1 = KT > 1 ? 1 : 0, k2 = KT > 2 ? 2 : KT - 1;
  load_b(0, 0, 0);
#pragma unroll
  for (int i = 0; i < 4; ++i) load_a(i, 0, 0);
#pragma unroll
  for (int j = 1; j < TN; ++j) load_b(j, 0, 0);
  load_b(0, 1, k1);
#pragma unroll
  for (int i = 0; i < 4; ++i) load_a(i, 1, k1);
  load_b(1, 1, k1);
  if constexpr (TN == 4) load_b(2, 1, k1);
  if constexpr (TN == 2) {
    load_b(0, 2, k2);
#pragma unroll
    for (int i = 0; i < 4; ++i) load_a(i, 2, k2);
  }
  wait_vmcnt_and_barrier<TN == 4 ? 10 : (TN == 3 ? 8 : 12)>();
  read_b(0, 0, 0);
  // (group 0 refills the region that these reads take from after this barrier)
  if (grp == 1) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  // LEFT: k-steps that follow, STAGES for as many or more; S: fragment set of block 0 (alternates where TN is odd).
  auto kstep = [&](int kt, auto set_c, auto left_c) __attribute__((always_inline)) {
    constexpr int S = decltype(set_c)::value, LEFT = decltype(left_c)::value;
    constexpr bool L1 = LEFT > 0, L2 = LEFT > 1, L3 = LEFT > 2;  // k-steps kt + 1, kt + 2, kt + 3 exist
    read_a(kt);
    if constexpr (TN == 4) {
      end_mem(DARE_N(L1 ? 9 : 2));
      matrix(0, 0, DARE_B(L1, 3, 1), none, DARE_B(L2, 0, 2), none);
      read_b(1, 1, kt);
      end_mem(DARE_N(L2 ? 10 : (L1 ? 9 : 1)));
      matrix(1, 1, DARE_A(L2, 0, 2), none, DARE_A(L2, 1, 2), none);
      read_b(0, 2, kt);
      end_mem(DARE_N(L2 ? 10 : (L1 ? 7 : 0)));
      matrix(0, 2, DARE_A(L2, 2, 2), none, DARE_A(L2, 3, 2), none);
      read_b(1, 3, kt);
      if constexpr (L1) read_b(0, 0, kt + 1);
      end_mem(DARE_N(L2 ? 8 : (L1 ? 3 : 0)));
      matrix(1, 3, DARE_B(L2, 1, 2), none, DARE_B(L2, 2, 2), none);
    } else if constexpr (TN == 2) {
      end_mem(DARE_N(L2 ? 10 : (L1 ? 5 : 0)));
      matrix(0, 0, DARE_B(L2, 1, 2), none, DARE_B(L3, 0, 3), none);
      read_b(1, 1, kt);
      if constexpr (L1) read_b(0, 0, kt + 1);
      end_mem(DARE_N(L3 ? 8 : (L2 ? 7 : (L1 ? 1 : 0))));
      matrix(1, 1, DARE_A(L3, 0, 3), DARE_A(L3, 1, 3), DARE_A(L3, 2, 3), DARE_A(L3, 3, 3));
    } else {
      end_mem(DARE_N(L1 ? 7 : 1));
      matrix(S, 0, DARE_B(L1, 2, 1), none, DARE_B(L2, 0, 2), none);
      read_b(S ^ 1, 1, kt);
      end_mem(DARE_N(L2 ? 7 : (L1 ? 6 : 0)));
      matrix(S ^ 1, 1, DARE_A(L2, 0, 2), DARE_A(L2, 1, 2), DARE_A(L2, 2, 2), DARE_A(L2, 3, 2));
      read_b(S, 2, kt);
      if constexpr (L1) read_b(S ^ 1, 0, kt + 1);
      end_mem(DARE_N(L2 ? 7 : (L1 ? 2 : 0)));
      matrix(S, 2, none, DARE_B(L2, 1, 2), none, none);
    }
  };
  // a k-step alone leaves the next one's block 0 in the set where it starts (branches that meet with different
  // sets cost registers)
  auto single = [&](int kt, auto left_c) __attribute__((always_inline)) {
    kstep(kt, DARE_N(0), left_c);
    if constexpr (TN == 3) {
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) fb[0][h][ks] = fb[1][h][ks];
    }
  };
  int kt = 0;
  if constexpr (TN == 3) {
    for (; kt + 1 < KT - STAGES; kt += 2) {
      kstep(kt, DARE_N(0), DARE_N(STAGES));
      kstep(kt + 1, DARE_N(1), DARE_N(STAGES));
    }
    if (kt < KT - STAGES) single(kt++, DARE_N(STAGES));
  } else {
    for (; kt < KT - STAGES; ++kt) kstep(kt, DARE_N(0), DARE_N(STAGES));
  }
  if constexpr (STAGES > 2) {
    if (kt < KT - 2) single(kt++, DARE_N(2));
  }
  if (kt < KT - 1) single(kt++, DARE_N(1));
  kstep(kt, DARE_N(0), DARE_N(0));
#undef DARE_N
#undef DARE_A
#undef DARE_B
  if (grp == 0) asm volatile("s_barrier" ::: "memory");
  wait_vmcnt<0>();

  // The workgroup that arrives last at a tile adds the other one's sums to its own (a sum of two
  // does not depend on which came first) and stores the tile; the other one leaves its sums in
  // its half of the tile's workspace and goes.  Nobody waits: a workgroup that finds the other's sums
  // complete need not store its own, and of two that both stored theirs the second one counted is
  // the last (1 us more per launch than a wait for the first one's sums).  The counter's
  // parity says whether one has arrived: even between launches, whatever the launch before left.
  // The sums are written and read at device scope (sc1: past whatever an XCD's L2 holds), and counted
  // once every wave's stores have completed, so no fence, which would write back the whole L2
  // (20-40 us), is needed.
  if constexpr (SPLIT) {
    constexpr int kDeviceScope = 16;  // cache policy sc1
    float* slots = p.split_tiles + (long)tile * (PARTS * BM * BN);
    const auto mine = __builtin_amdgcn_make_buffer_rsrc(slots + (unit & 1) * (BM * BN), 0, BM * BN * 4, 0x00027000);
    const auto other = __builtin_amdgcn_make_buffer_rsrc(slots + (~unit & 1) * (BM * BN), 0, BM * BN * 4, 0x00027000);
    int* count = p.split_count + tile;
    int* last = reinterpret_cast<int*>(smem);
    __syncthreads();
    if (tid == 0) *last = __hip_atomic_load(count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & 1;
    __syncthreads();
    if (!*last) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2 * TN; ++j)
          __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, acc[i][j]), mine,
                                                 ((i * 2 * TN + j) * 512 + tid) * 16, 0, kDeviceScope);
      wait_vmcnt<0>();
      __syncthreads();
      if (tid == 0) *last = __hip_atomic_fetch_add(count, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & 1;
      __syncthreads();
      if (!*last) return true;
    } else if (tid == 0) {
      __hip_atomic_fetch_add(count, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 2 * TN; ++j)
        acc[i][j] += __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                                   other, ((i * 2 * TN + j) * 512 + tid) * 16, 0, kDeviceScope));
  }

  // acc[i][2 j + h][e] = C[row, col], row = m0 + 64 wm + 16 i + l16, col = n0 + 32 TN grp + 32 j + 8 kq + 4 h + e
  int col[TN];
#pragma unroll
  for (int j = 0; j < TN; ++j) col[j] = n0 + grp * (32 * TN) + j * 32 + kq * 8;
  store_tile<8>(p, p.c32, tok_out, live_out, col, [&](int i, int j, int e) __attribute__((always_inline)) {
    return acc[i][j * 2 + (e >> 2)][e & 3];
  });
  return true;
}

// ---- several rounds of large tiles of all rows: 256 x (64 TN), four waves, one per SIMD ----
// A wave owns 128 rows x 32 TN columns, its sums in the accumulator registers, which leaves the others to two sets of
// fragments: a slice of 32 k is multiplied while the next one's fragments are read.  Against gemm_tile_pp, whose eight waves take 64
// rows each: a third fewer bytes read from LDS per k-step (131 KB for 196), one barrier for eight, and what these kernels are bound
// by, power, goes with both (a 256 x 256 tile with 192 k-steps, random operands: 278 us, without the loads into LDS 224, without the
// fragment reads 250, with neither 201).
//   * One instruction stream.  A read every three MFMAs, a load every eight (TN = 4), the address of a load one MFMA later, nothing
//     between two MFMAs that takes longer than one.  The MFMAs are inline assembly: the compiler, which may put the sums into either kind of
//     registers, moved 400 of them per k-step.  It does not know these as MFMAs, so their results wait by hand (s_nop).
//   * LDS: half-stages A(0), B(0), A(1), B(1), .. of a k-step each through a ring of five slots, 160 KB.  The barrier of a
//     k-step lies between its two slices: every wave has read A(kt) and B(kt), and A(kt + 1) and B(kt + 1) have landed.  In front of
//     it A(kt + 2) is loaded (into the slot of B(kt - 1)), behind it B(kt + 2) (into that of A(kt)): a load has one to three
//     slices of 1024 cycles to arrive; never waiting for any is no faster.
//   * The pipeline runs on from tile to tile: a workgroup per CU walks its tiles, the last two k-steps load the next tile's
//     first two and the last slice reads its first fragments, so a tile ends without an empty ring.  Behind the last tile they
//     load their own k-steps again, into slots that nobody reads: the same code, where code of its own for the end and the start, fetched
//     once per launch, cost a launch of one round 3 us.
//   * Stores of whole 128-byte lines: rows 0 .. 7 of a block of 16 in one store and 8 .. 15 in the next, two column blocks side
//     by side (lanes L and L ^ 8 swap halves).  Stores count in vmcnt with the loads, in order, and the loads of the next tile
//     wait for them: with 64-byte runs they took 9 us per round of the CUs.
// The sum over k is formed as in gemm_tile_pp and gemm_tile16, so results are the same bits.
// us, gemm_tile_pp (256 x 192 and 256) and now, one card: 16384 x 12288 x 4096 1148 and 1076 (1.53 PFLOP/s), 16384 x 4096 x 4096 384 and 362,
// 4096 x 24576 x 4096 608 and 541, 4096 x 4096 x 12288 272 and 262, 2331 x 12288 x 4096 184 and 177, with operands in the caches.
// In steps, where they come from other kernels and from memory: 4096 x 24576 with
// the gate 570 and 547, 8192 x 24576 1123 and 1079, 4096 x 4096 x 12288 277 and 270, Q, K and V of 4096 rows, rotated, 314 and 297;
// one round is better off with eight waves (four_waves, gemm_route.h).
// The gate of 128 x 128 sums takes a wave 2.8 us (with the compiler's division 5.5), the rotation 2.
// gemm_tile_pp stays for 256 x 128 (gemm_bf16_pp_kernel), for one round, where k is cut over two workgroups (1024 x 4096 x 12288 92.6 us, in this form 103.6: half as many waves store and add
// the sums) and for listed rows, whose kernel has the eight waves that the small shapes want.
constexpr int kQuadSlot = kPpRows * ROW_BYTES, kQuadSmem = 5 * kQuadSlot;

// Value of a lane from the lane 8 further on in its row of 16, in the lanes of BANKS (four lanes each); `own` in the others
template <int BANKS>
__device__ __forceinline__ unsigned from_half_row(unsigned own, unsigned other) {
  return __builtin_amdgcn_update_dpp(own, other, 0x128, 0xf, BANKS, false);
}
// STREAM: past the L2
template <bool STREAM>
__device__ __forceinline__ void store16(bf16_t* to, const u32x4 v) {
  if constexpr (STREAM)
    __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(to));
  else
    *reinterpret_cast<u32x4*>(to) = v;
}

// The tiles blockIdx.x, blockIdx.x + gridDim.x, ..; called by all 256 threads.  k of kQuadMinSteps k-steps or more (loads two ahead, and
// the first one's zero sums).
// PART: the columns from part_n on for all rows, those in front of it for the part_m rows of the second list.
template <int TN, bool STREAM, bool PART = false>
__device__ __forceinline__ void gemm_tiles_quad(const GemmDev& p, const int m, unsigned char* smem, const int part_m = 0) {
  static_assert(TN == 3 || TN == 4, "column blocks of 32 per wave");
  constexpr int BM = kPpRows, BN = 64 * TN;
  constexpr int SLOT = kQuadSlot;
  constexpr int AL = BM / 8 / 4, BL = BN / 8 / 4;  // loads of a wave per half-stage
  constexpr int NA = 8, NB = 2 * TN;               // fragments of a slice
  constexpr int NM = NA * NB, NR = NA + NB;        // its MFMAs and reads

  const int first_n = PART ? p.part_n : 0;
  const int tiles_m = (m + BM - 1) / BM, tiles_n = (p.n - first_n + BN - 1) / BN, all = tiles_m * tiles_n;
  const int part_tiles_m = (part_m + BM - 1) / BM, part_tiles_n = (first_n + BN - 1) / BN;
  const int total = all + part_tiles_m * part_tiles_n;
  const int per_xcd = (total + 7) >> 3;
  int vb = blockIdx.x, m0, n0;
  int rows_end = m, cols_end = p.n;     // of the tile's list and columns
  const int32_t* list = p.idx;
  auto place = [&]() __attribute__((always_inline)) {
    const int slot = vb >> 3, unit = (vb & 7) * per_xcd + slot;
    if (slot >= per_xcd || unit >= total) return false;
    int tile_m, tile_n;
    if (!PART || unit < all) {
      tile_of_unit(unit, tiles_m, tiles_n, tile_m, tile_n);
      n0 = first_n + tile_n * BN;
    } else {
      tile_of_unit(unit - all, part_tiles_m, part_tiles_n, tile_m, tile_n);
      n0 = tile_n * BN;
      rows_end = part_m;
      cols_end = first_n;
      list = p.part_idx;
    }
    m0 = tile_m * BM;
    return true;
  };
  if (!place()) return;

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave & 1, wn = wave >> 1;
  const int l16 = lane & 15, kq = lane >> 4;
  const int KT = p.k / BK;

  // the rows of this lane's loads
  int tok_in[AL];
  auto rows = [&]() __attribute__((always_inline)) {
    int row_in[AL];
#pragma unroll
    for (int i = 0; i < AL; ++i) {
      const int row = m0 + (wave * AL + i) * 8 + (lane >> 3);
      row_in[i] = row < rows_end ? row : rows_end - 1;
    }
    row_tokens(list, nullptr, row_in, tok_in);
  };
  const bf16_t* src_a[AL];
  const bf16_t* src_b[BL];
  auto addresses = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < AL; ++i) {
      const int r = (wave * AL + i) * 8 + (lane >> 3);
      src_a[i] = p.a + (long)tok_in[i] * p.lda + ((lane & 7) ^ ((r >> 1) & 7)) * 8;
    }
#pragma unroll
    for (int j = 0; j < BL; ++j) {
      const int r = (wave * BL + j) * 8 + (lane >> 3);
      const int col = n0 + r < cols_end ? n0 + r : cols_end - 1;
      src_b[j] = p.wt + (long)col * p.k + ((lane & 7) ^ pp_bkey(r & 31)) * 8;
    }
  };
  const unsigned lds0 = (unsigned)(size_t)(lptr_t)smem;
  // (the address is an operand in M0, set by the compiler, which then knows what M0 holds; a wait state, or an MFMA,
  // between the move to M0 and the load)
  auto load = [&](const bf16_t*& src, unsigned lds) __attribute__((always_inline)) {
    asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(src), "{m0}"(lds) : "memory");
    src += BK;
  };

  f32x4 acc[NA][NB];
  int a_off[2], b_off[2];
  const int brow = (l16 >> 2) * 8 + (l16 & 3);
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) {
    a_off[ks] = (wm * 128 + l16) * ROW_BYTES + ((ks * 4 + kq) ^ ((l16 >> 1) & 7)) * 16;
    b_off[ks] = (wn * 32 * TN + brow) * ROW_BYTES + ((ks * 4 + kq) ^ pp_bkey(brow)) * 16;
  }
  bf16x8 fa[2][NA], fb[2][NB];
  typedef const __attribute__((address_space(3))) bf16x8* lds_frag_t;
  // read n of a slice: the first column's fragment, the rows', the other columns'
  auto read = [&](auto ks_c, int n, unsigned at_a, unsigned at_b) __attribute__((always_inline)) {
    constexpr int ks = decltype(ks_c)::value;
    if (n >= 1 && n <= NA)
      fa[ks][n - 1] = *(lds_frag_t)(at_a + (n - 1) * 16 * ROW_BYTES);
    else {
      const int j = n == 0 ? 0 : n - NA;
      fb[ks][j] = *(lds_frag_t)(at_b + (j >> 1) * 32 * ROW_BYTES + (j & 1) * 4 * ROW_BYTES);
    }
  };
  // the MFMAs of a slice with the next slice's reads and the loads of a half-stage between them
  auto slice = [&](auto ks_c, auto zero_c, auto n_loads, const bf16_t** src, unsigned to, int at_a, int at_b) __attribute__((always_inline)) {
    constexpr int ks = decltype(ks_c)::value, NL = decltype(n_loads)::value;
    const unsigned ra = lds0 + at_a + a_off[ks ^ 1], rb = lds0 + at_b + b_off[ks ^ 1];
    constexpr int RS = NM / NR < 3 ? NM / NR : 3, LS = NM / NL;  // MFMAs per read, per load
    static_assert(RS * NR <= NM && LS > 3, "every fragment must have its read, every load its place");
#pragma unroll
    for (int t = 0; t < NM; ++t) {
      const int j = t / NA, i = t % NA;
      const int l = t / LS;
      const bool loads = t % LS == 2 && l < NL;
      if constexpr (decltype(zero_c)::value) {
        if (loads)
          asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0\n\tglobal_load_lds_dwordx4 %3, off" : "=a"(acc[i][j]) : "v"(fb[ks][j]), "v"(fa[ks][i]), "v"(src[l]), "{m0}"(to + l * 1024) : "memory");
        else
          asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=a"(acc[i][j]) : "v"(fb[ks][j]), "v"(fa[ks][i]));
      } else {
        if (loads)
          asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0\n\tglobal_load_lds_dwordx4 %3, off" : "+a"(acc[i][j]) : "v"(fb[ks][j]), "v"(fa[ks][i]), "v"(src[l]), "{m0}"(to + l * 1024) : "memory");
        else
          asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc[i][j]) : "v"(fb[ks][j]), "v"(fa[ks][i]));
      }
      __builtin_amdgcn_sched_barrier(0);
      if (t % RS == 0 && t / RS < NR) {
        read(std::integral_constant<int, ks ^ 1>{}, t / RS, ra, rb);
        __builtin_amdgcn_sched_barrier(0);
      }
      if (t % LS == 3 && l < NL) {  // (next to an MFMA of its own)
        src[l] += BK;
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
#define DARE_N(n) std::integral_constant<int, n>{}
  using Yes = std::true_type;
  using No = std::false_type;
  auto wrap = [](int at) __attribute__((always_inline)) { return at >= 5 * SLOT ? at - 5 * SLOT : at; };
  int at = 0;  // slot of A(kt)
  auto kstep = [&](auto zero_c) __attribute__((always_inline)) {
    const int b0 = wrap(at + SLOT), a1 = wrap(at + 2 * SLOT), b1 = wrap(at + 3 * SLOT), a2 = wrap(at + 4 * SLOT);
    slice(DARE_N(0), zero_c, DARE_N(AL), src_a, lds0 + a2 + wave * AL * 1024, at, b0);
    wait_vmcnt_and_barrier<AL>();
    __builtin_amdgcn_sched_barrier(0);
    slice(DARE_N(1), No{}, DARE_N(BL), src_b, lds0 + at + wave * BL * 1024, a1, b1);
    at = a1;
  };

  rows();
  addresses();
#pragma unroll
  for (int k = 0; k < 2; ++k) {
#pragma unroll
    for (int i = 0; i < AL; ++i) load(src_a[i], lds0 + 2 * k * SLOT + (wave * AL + i) * 1024);
#pragma unroll
    for (int j = 0; j < BL; ++j) load(src_b[j], lds0 + (2 * k + 1) * SLOT + (wave * BL + j) * 1024);
  }
#pragma unroll
  for (int i = 0; i < NA; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
      asm volatile("" : "+a"(acc[i][j]));
    }
  wait_vmcnt_and_barrier<AL + BL>();
#pragma unroll
  for (int n = 0; n < NR; ++n) read(DARE_N(0), n, lds0 + a_off[0], lds0 + SLOT + b_off[0]);
  __builtin_amdgcn_sched_barrier(0);
  for (int kt = 0;;) {
    int row_out[NA], tok[NA];
    bool live[NA];
#pragma unroll
    for (int i = 0; i < NA; ++i) {
      const int row = m0 + wm * 128 + i * 16 + l16;
      live[i] = row < rows_end;
      row_out[i] = row < rows_end ? row : rows_end - 1;
    }
    row_tokens(list, nullptr, row_out, tok);
    const int col0 = n0 + wn * (32 * TN), n_end = cols_end;
    vb += gridDim.x;
    const bool more = place();
    if (more) rows();
    for (; kt < KT; ++kt) {
      if (kt == KT - 2) {
        if (more) {
          addresses();
        } else {  // the last two k-steps again, into slots that nobody reads
#pragma unroll
          for (int i = 0; i < AL; ++i) src_a[i] -= 2 * BK;
#pragma unroll
          for (int j = 0; j < BL; ++j) src_b[j] -= 2 * BK;
        }
      }
      kstep(No{});
    }
    // (what the compiler would know of MFMAs of its own: their results are there 18 cycles later)
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
    auto value = [&](int i, int j, int e) __attribute__((always_inline)) {
      float v;
      asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(v) : "a"(acc[i][j * 2 + (e >> 2)][e & 3]));
      return v;
    };
    // acc[i][2 j + h][e] = C[row, col], row = m0 + 128 wm + 16 i + l16, col = col0 + 32 j + 8 kq + 4 h + e
    const bool low = l16 < 8;
    if (!PART && p.swiglu_pairs) {
      const long ldc = p.ldc;
#pragma unroll
      for (int i = 0; i < NA; ++i) {
        u32x2 o[TN];
        float q[TN][4];
        unsigned lowest = 0;  // as bits: of two negative floats the lower one has the larger bits
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float g = value(i, j, 2 * e);
            lowest = max(lowest, __float_as_uint(g));
            q[j][e] = silu<false>(g);
          }
        // (scaled where some lane needs it: scaling every gate made model steps of 1430, 3609 and 3940 us 12, 16 and 19 us longer;
        // traced, 1024 x 24576 x 4096 with the gate takes 149.8 us without this and 149.5 with it)
        if (__builtin_expect(__any(lowest > __float_as_uint(kGateLow)), 0)) {
#pragma unroll
          for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) q[j][e] = silu(value(i, j, 2 * e));
        }
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          bf16x4 r;
#pragma unroll
          for (int e = 0; e < 4; ++e) r[e] = (bf16_t)(q[j][e] * value(i, j, 2 * e + 1));
          o[j] = __builtin_bit_cast(u32x2, r);
        }
        // lanes kq and kq ^ 1 share two column blocks: 16 bytes of one of them each
        u32x4 w[TN / 2];
#pragma unroll
        for (int j = 0; j + 1 < TN; j += 2)
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            const auto sw = __builtin_amdgcn_permlane16_swap(o[j][q], o[j + 1][q], false, false);
            w[j / 2][q] = sw[0];
            w[j / 2][q + 2] = sw[1];
          }
        bf16_t* own = p.c0 + tok[i] * ldc + (col0 >> 1);
        const int at_col = (kq & 1) * 16 + (kq >> 1) * 8;
        if constexpr (TN == 4) {
          const int other = from_half_row<0xf>(0, tok[i]);
          const bool live_other = from_half_row<0xf>(0, live[i]) != 0;
          u32x4 x, y;
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            x[q] = from_half_row<0xc>(w[0][q], w[1][q]);
            y[q] = from_half_row<0x3>(w[1][q], w[0][q]);
          }
          bf16_t* far = p.c0 + other * ldc + (col0 >> 1);
          const int c = at_col + (low ? 0 : 32);
          const bool in = col0 + (low ? 0 : 64) < n_end;
          if (in && (low ? live[i] : live_other)) store16<STREAM>((low ? own : far) + c, x);
          if (in && (low ? live_other : live[i])) store16<STREAM>((low ? far : own) + c, y);
        } else {
          if (live[i] && col0 + (kq & 1) * 32 < n_end) store16<STREAM>(own + at_col, w[0]);
          if (live[i] && col0 + 64 < n_end) *reinterpret_cast<u32x2*>(own + 32 + kq * 4) = o[TN - 1];
        }
      }
    } else {
      if (!PART && p.c32 && col0 < p.c32_cols) {
#pragma unroll
        for (int i = 0; i < NA; ++i)
#pragma unroll
          for (int j = 0; j < NB; ++j) {
            const int c = col0 + (j >> 1) * 32 + kq * 8 + (j & 1) * 4;
            f32x4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = value(i, j >> 1, (j & 1) * 4 + e);
            if (live[i] && c < p.c32_cols) *reinterpret_cast<f32x4*>(p.c32 + (long)tok[i] * p.c32_cols + c) = v;
          }
      }
      if (p.rope && col0 < p.rope_cols) {
        // (the table's rows a row of the tile ahead of their use; columns that are not rotated read one that is)
        f32x4 cs[2][NB];
        auto table = [&](int i) __attribute__((always_inline)) {
          const float* row = p.rope + (long)((unsigned)tok[i] % (unsigned)p.rope_seq) * p.rope_dh;
#pragma unroll
          for (int j = 0; j < NB; ++j) {
            const int c = col0 + (j >> 1) * 32 + kq * 8 + (j & 1) * 4;
            cs[i & 1][j] = *reinterpret_cast<const f32x4*>(row + ((unsigned)(c < p.rope_cols ? c : col0) % (unsigned)p.rope_dh >> 1) * 2);
          }
        };
        table(0);
#pragma unroll
        for (int i = 0; i < NA; ++i) {
          if (i + 1 < NA) table(i + 1);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int j = 0; j < NB; ++j) {
            const bool turns = col0 + (j >> 1) * 32 + kq * 8 + (j & 1) * 4 < p.rope_cols;
            float v[4], w[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = w[e] = value(i, j >> 1, (j & 1) * 4 + e);
            rope_rotate4(cs[i & 1][j], w[0], w[1], w[2], w[3]);
            acc[i][j] = f32x4{turns ? w[0] : v[0], turns ? w[1] : v[1], turns ? w[2] : v[2], turns ? w[3] : v[3]};
            asm volatile("" : "+a"(acc[i][j]));
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      // the column blocks' places: a pair's first block in the lanes of rows 0 .. 7, its second one in the others
      bf16_t* base[(TN + 1) / 2];
#pragma unroll
      for (int j = 0; j < TN; j += 2) {
        const int c = col0 + j * 32 + (j + 1 < TN && !low ? 32 : 0);
        const int seg = (c >= p.seg_n) + (c >= 2 * p.seg_n);
        bf16_t* to = c >= n_end ? nullptr : seg == 0 ? p.c0 : seg == 1 ? p.c1 : p.c2;
        base[j / 2] = to ? to + (c - seg * p.seg_n) + kq * 8 : nullptr;
      }
      const long ldc = p.ldc;
#pragma unroll
      for (int i = 0; i < NA; ++i) {
        const int other = from_half_row<0xf>(0, tok[i]);
        const bool live_other = from_half_row<0xf>(0, live[i]) != 0;
        const long own = tok[i] * ldc, far = other * ldc;
#pragma unroll
        for (int j = 0; j < TN; j += 2) {
          u32x4 o[2];
#pragma unroll
          for (int h = 0; h < 2; ++h)
            if (j + h < TN) {
              bf16x8 r;
#pragma unroll
              for (int e = 0; e < 8; ++e) r[e] = (bf16_t)value(i, j + h, e);
              o[h] = __builtin_bit_cast(u32x4, r);
            }
          bf16_t* to = base[j / 2];
          if (j + 1 < TN) {
            u32x4 x, y;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              x[q] = from_half_row<0xc>(o[0][q], o[1][q]);
              y[q] = from_half_row<0x3>(o[1][q], o[0][q]);
            }
            if (to && (low ? live[i] : live_other)) store16<STREAM>(to + (low ? own : far), x);
            if (to && (low ? live_other : live[i])) store16<STREAM>(to + (low ? far : own), y);
          } else if (to && live[i]) {
            store16<STREAM>(to + own, o[0]);
          }
        }
      }
    }
    if (!more) break;
    kstep(Yes{});
    kt = 1;
  }
#undef DARE_N
  wait_vmcnt<0>();
}

// Columns [0, part_n) for the listed rows, whose count the device knows, and the others for all rows: one launch for
// both, in the shape of the least cost.  Two shapes, no gate and no fp32 copy: 8310 instructions and no spilled scalar, where 256 x 128, which
// is slower with the weights in memory, and those epilogues made it 22345 and 38 (block steps, with them and without, us: 5 x 1024 tokens
// of hidden 4096, a twentieth refreshed, 403.8 400.7, 4 x 800 half refreshed 385.4 383.3, 16 x 1000 of hidden 2048 392.0 385.9).
__global__ void __launch_bounds__(256, 1) gemm_bf16_part_kernel(GemmDev p) {
  __shared__ __attribute__((aligned(1024))) unsigned char smem[kQuadSmem];
  const int part_m = *(const __attribute__((address_space(4))) int32_t*)(uintptr_t)p.part_m_dev;
  if (part_columns(p.m_max, p.n, part_m, p.part_n) == 3) return gemm_tiles_quad<3, false, true>(p, p.m_max, smem, part_m);
  gemm_tiles_quad<4, false, true>(p, p.m_max, smem, part_m);
}

template <int TN, bool STREAM>
__global__ void __launch_bounds__(256, 1) gemm_bf16_quad_kernel(GemmDev p) {
  __shared__ __attribute__((aligned(1024))) unsigned char smem[kQuadSmem];
  gemm_tiles_quad<TN, STREAM>(p, p.m_max, smem);
}

// ---- very few rows (at most 16 TMS): a stream over the weight matrix ------------------
// With a handful of refreshed rows (one or two tokens unmasked per denoising step) the
// projection is a matrix-vector product in disguise: what matters is that every CU pulls on
// the weight stream at once and that each weight byte is read once.  A workgroup owns 16
// output columns for the whole of k; its NW waves take contiguous ranges of k, load their
// weight and row fragments straight into registers (no LDS: a fragment is used by one wave
// only), 16 k-steps of 32 in flight per wave (8 with two row blocks), multiply with v_mfma_f32_16x16x32_bf16
// (weight fragment first, so a lane again owns one row and four neighbouring columns), and
// the partial sums of the waves are added in wave order through LDS.
template <int NW, int TMS>
__device__ __forceinline__ void skinny_tile(const GemmDev& p, const int m, unsigned char* smem, const int tid,
                                            lds_idx_t lidx = nullptr) {
  constexpr int UNR = TMS == 1 ? 16 : 8;
  // (the wave number as a scalar: LDS addresses of the global -> LDS loads go through M0, and a
  // wave number held in a vector register would send every one of them through v_readfirstlane)
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, kq = lane >> 4;
  const int groups = p.n >> 4;
  const int steps = p.k >> 5;
  const int spw = (steps + NW - 1) / NW;
  const int s0 = wave * spw;
  const int s1 = s0 + spw < steps ? s0 + spw : steps;
  const bf16_t* xrow[TMS];
  int row[TMS], tok[TMS];
  bool live[TMS];
#pragma unroll
  for (int t = 0; t < TMS; ++t) {
    live[t] = t * 16 + l16 < m;
    row[t] = live[t] ? t * 16 + l16 : m - 1;
  }
  row_tokens(p.idx, lidx, row, tok);
#pragma unroll
  for (int t = 0; t < TMS; ++t) xrow[t] = p.a + (long)tok[t] * p.lda + kq * 8;
  f32x4* red = reinterpret_cast<f32x4*>(smem);  // [NW][TMS][64]
  for (int grp = blockIdx.x; grp < groups; grp += gridDim.x) {
    const int n0 = grp << 4;
    const bf16_t* wrow = p.wt + (long)(n0 + l16) * p.k + kq * 8;
    f32x4 acc[TMS];
#pragma unroll
    for (int t = 0; t < TMS; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int s = s0; s < s1; s += UNR) {
      bf16x8 wf[UNR], xf[TMS][UNR];
#pragma unroll
      for (int u = 0; u < UNR; ++u) {
        const bool live = s + u < s1;
        const int ks = (live ? s + u : s0) << 5;
        wf[u] = *reinterpret_cast<const bf16x8*>(wrow + ks);
#pragma unroll
        for (int t = 0; t < TMS; ++t) xf[t][u] = *reinterpret_cast<const bf16x8*>(xrow[t] + ks);
        if (!live) {
#pragma unroll
          for (int e = 0; e < 8; ++e) wf[u][e] = (bf16_t)0.0f;
        }
      }
#pragma unroll
      for (int u = 0; u < UNR; ++u)
#pragma unroll
        for (int t = 0; t < TMS; ++t)
          acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[u], xf[t][u], acc[t], 0, 0, 0);
    }
    // (the wait for the MFMAs by hand: the compiler, which has to put it in front of the stores, left it out
    // here, behind a loop that a second path goes round, and three of four columns were stored too early)
#pragma unroll
    for (int t = 0; t < TMS; ++t) asm volatile("s_nop 7\n\ts_nop 1" : "+v"(acc[t]));
#pragma unroll
    for (int t = 0; t < TMS; ++t) red[(wave * TMS + t) * 64 + lane] = acc[t];
    __syncthreads();
    if (wave == 0) {
#pragma unroll
      for (int t = 0; t < TMS; ++t) {
        acc[t] = red[t * 64 + lane];
        for (int w = 1; w < NW; ++w) acc[t] += red[(w * TMS + t) * 64 + lane];
      }
      const int col[1] = {n0 + kq * 4};
      store_tile<4>(p, p.c32, tok, live, col,
                    [&](int t, int, int e) __attribute__((always_inline)) { return acc[t][e]; });
    }
    __syncthreads();
  }
}
constexpr int kSkinnyRows = 32, kSkinnyMaxN = 8192;

// ---- one tile shape, chosen on the host (row count known): k in ranges, then whole k --------------
template <int BM, int BN, int WAVES_M, int WAVES_N, int STAGES>
__global__ void __launch_bounds__(WAVES_M* WAVES_N * 64) gemm_bf16_ranges_kernel(GemmDev p) {
  __shared__ __attribute__((aligned(1024))) unsigned char smem[smem_bytes<BM, BN, STAGES>()];
  gemm_tile<BM, BN, WAVES_M, WAVES_N, STAGES>(p, p.m_max, smem);
}

template <int BM, int BN, int WAVES_M, int WAVES_N, int STAGES>
__global__ void __launch_bounds__(512) gemm_bf16_tile16_kernel(GemmDev p) {
  __shared__ __attribute__((aligned(1024))) unsigned char smem[smem_bytes<BM, BN, STAGES>()];
  gemm_tile16<BM, BN, WAVES_M, WAVES_N, STAGES>(p, p.m_max, smem, threadIdx.x, blockIdx.x);
}

// All rows: 256 x 128, and a round of 256 x 192 or 256 (four_waves, gemm_route.h).  256 x 128: with the weights in memory eight waves and
// three stages in flight are faster than four waves, whose ring holds two and a half: 1320 x 3072 x 9216 102 us and 119, x 3072 x 3072
// 39-44 and 45-52 (in the caches 91.6 and 83.4, 34.9 and 33.2).
template <int TN, bool SPLIT>
__global__ void __launch_bounds__(512) gemm_bf16_pp_kernel(GemmDev p) {
  __shared__ __attribute__((aligned(1024))) unsigned char smem[pp_smem_bytes<TN>()];
  gemm_tile_pp<TN, SPLIT>(p, p.m_max, smem, blockIdx.x);
}

// ---- row count read on the device: the tile shape follows it -------------------------
// One kernel for every projection of refreshed rows that has a choice of shapes, 8 waves and 144 KiB of LDS, one workgroup per CU
// whatever the count turns out to be (a grid sized for the worst case, whose surplus workgroups
// return at once, costs 1 us more at 205 rows); the shape is the one that best_tile (gemm_route.h) names, and
// its tiles are walked in passes.
constexpr int kWideSmem = pp_smem_bytes<2>();
constexpr int kWideGrid = 256;  // workgroups of a launch: one per CU
// The refreshed-row list from the mask bytes, by every workgroup for itself (Alg. 1/2 line 5
// folded into the first kernel that needs the list: a compaction kernel of its own costs a
// launch, 4-5 us of a 90 us step, for a few hundred bytes of work).  512 threads, up to
// kSelMaxTokens tokens, four per thread; ascending by construction.  Returns the count.
// While the mask is on its way and the list is made, the first 256 k of the weight rows are read ahead: an XCD's
// workgroups, 16 rows each at a time, read its share of them (tiles are dealt to the XCDs in contiguous ranges of
// columns, as long as there are at most GROUP_M row tiles) into its L2, into 1 KiB of LDS that nobody reads; nothing here
// waits for them.  What it fills is the time of the mask's round trip and the list.  (The first
// one in a block with the mask: the compiler waits for loads into LDS with those in front of them.)  Steps over 1 x 1024
// tokens with 205 refreshed rows, without and with it (us): hidden 4096 89.2 and 87.7, 6144 155.7 and 154.0, 1024 to 3072 and
// 8192, and 4 rows, no difference beyond the runs'.  The stream over the weights (skinny_tile) deals its columns
// otherwise and has nothing from it.
__device__ __forceinline__ int derive_rows(const GemmDev& p, int32_t* list, int* wave_tot, unsigned char* nobody) {
  const int n_tok = p.sel_batch * p.sel_seq;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int t0 = tid * 4;
  const int per_xcd = (p.n + 7) >> 3, first = (blockIdx.x & 7) * per_xcd, slots = gridDim.x >> 3;
  const int last = first + per_xcd < p.n ? first + per_xcd - 1 : p.n - 1;
  const uint8_t* mask[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) mask[k] = p.sel_mask + (t0 + k < n_tok ? t0 + k : n_tok - 1);
  auto ahead = [&](int i) __attribute__((always_inline)) {
    const int r = first + (((blockIdx.x >> 3) + i * slots) * 8 + wave) * 2 + (lane >> 5);
    return p.wt + (long)(r < last ? r : last) * p.k + ((lane & 31) * 8 < p.k ? (lane & 31) * 8 : 0);
  };
  const unsigned lds = (unsigned)(size_t)(lptr_t)nobody;
  int reused[4];
  asm volatile(
      "global_load_ubyte %0, %4, off\n\tglobal_load_ubyte %1, %5, off\n\t"
      "global_load_ubyte %2, %6, off\n\tglobal_load_ubyte %3, %7, off\n\t"
      "global_load_lds_dwordx4 %8, off\n\ts_waitcnt vmcnt(1)"
      : "=&v"(reused[0]), "=&v"(reused[1]), "=&v"(reused[2]), "=&v"(reused[3])
      : "v"(mask[0]), "v"(mask[1]), "v"(mask[2]), "v"(mask[3]), "v"(ahead(0)), "{m0}"(lds)
      : "memory");
#pragma unroll 1
  for (int i = 1; i < p.ahead; ++i)
    asm volatile("global_load_lds_dwordx4 %0, off" ::"v"(ahead(i)), "{m0}"(lds) : "memory");
  bool z[4];
  int cnt = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    z[k] = t0 + k < n_tok && reused[k] == 0;
    cnt += z[k];
  }
  int incl = cnt;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int up = __shfl_up(incl, o, 64);
    if (lane >= o) incl += up;
  }
  if (lane == 63) wave_tot[wave] = incl;
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  int rank = incl - cnt, total = 0;
#pragma unroll
  for (int w = 0; w < 8; ++w) {
    if (w < wave) rank += wave_tot[w];
    total += wave_tot[w];
  }
#pragma unroll
  for (int k = 0; k < 4; ++k)
    if (z[k]) list[rank++] = t0 + k;
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  if (blockIdx.x == 0) {  // what the compaction kernel would have written, for the kernels that follow
    for (int r = tid; r < total; r += 512) {
      p.sel_idx_out[r] = list[r];
      if (p.sel_idx_out2) p.sel_idx_out2[r] = list[r];
    }
    // refreshed tokens in front of sequence b: first list position holding a token >= b * seq
    auto before = [&](int b) {
      const int key = b * p.sel_seq;
      int lo = 0, hi = total;
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (list[mid] < key) lo = mid + 1; else hi = mid;
      }
      return lo;
    };
    for (int b = tid; b <= p.sel_batch; b += 512) {  // (a batch may have more sequences than threads)
      const int off = before(b);
      p.sel_off_out[b] = off;
      if (p.sel_count_out && b < p.sel_batch) p.sel_count_out[b] = before(b + 1) - off;
    }
  }
  return total;
}

// The count of listed rows and, FUSED, the list derived from the mask bytes inside the kernel (two instantiations,
// so that the plain one carries none of the list handling), behind STAGES bytes of stage memory: 64 bytes of sums, the
// list, 1 KiB that nobody reads; else that KiB alone.
template <bool FUSED>
constexpr int kListBytes = FUSED ? 64 + kSelMaxTokens * 4 + 1024 : 1024;
template <bool FUSED, int STAGES>
__device__ __forceinline__ int listed_rows(const GemmDev& p, unsigned char* smem, lds_idx_t& lidx) {
  if constexpr (FUSED) {
    int32_t* list = reinterpret_cast<int32_t*>(smem + STAGES + 64);
    const int m = derive_rows(p, list, reinterpret_cast<int*>(smem + STAGES), smem + STAGES + 64 + kSelMaxTokens * 4);
    lidx = (lds_idx_t)list;
    return m;
  } else {
    // (the weights ahead as in derive_rows, 16 rows per workgroup: the count and the list are a shorter wait, and the
    // list, which comes behind these loads, must not wait for more.  Steps over 1 x 1024 tokens with 205 refreshed rows, hidden
    // 1024 40.9 -> 40.6 us, 3072 70.8 -> 70.2, 4096 87.7 -> 86.9; with 4 rows, the stream, no difference; 16384 tokens unchanged)
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int per_xcd = (p.n + 7) >> 3, first = (blockIdx.x & 7) * per_xcd;
    const int last = first + per_xcd < p.n ? first + per_xcd - 1 : p.n - 1;
    const int r = first + ((blockIdx.x >> 3) * 8 + wave) * 2 + (lane >> 5);
    const bf16_t* ahead = p.wt + (long)(r < last ? r : last) * p.k + ((lane & 31) * 8 < p.k ? (lane & 31) * 8 : 0);
    __builtin_amdgcn_global_load_lds((gptr_t)ahead, (lptr_t)(smem + STAGES), 16, 0, 0);
    // (a scalar load, which does not wait for the weights)
    return p.m_dev ? *(const __attribute__((address_space(4))) int32_t*)(uintptr_t)p.m_dev : p.m_max;
  }
}
// Up to 32 rows and a narrow output (the output projection): the register-fed stream
// (measured at n = 4096: 11-15 us against 17 us for 64 x 64 tiles, which give that width
// only 64 workgroups).  Wide outputs keep the 64 x 64 tiles for few rows: with 192
// column tiles they already stream the weights at 5 TB/s.
__device__ __forceinline__ bool few_rows(const GemmDev& p, const int m, unsigned char* smem, lds_idx_t lidx) {
  if (m > kSkinnyRows || p.n >= kSkinnyMaxN) return false;
  if (m <= 16) skinny_tile<8, 1>(p, m, smem, threadIdx.x, lidx); else skinny_tile<8, 2>(p, m, smem, threadIdx.x, lidx);
  return true;
}

// Sizes that 64 x 64 tiles serve in one round whatever the count turns out to be: without the other shapes and the rule (what
// bounds such a launch is its own start: code fetched once, the list, the first reads).  Launches of 80 rows, 402 x 1536 x 512 and 402 x
// 512 x 512, with the kernel of all shapes and with this one 5.48 and 5.14, 5.44 and 5.12 us; a step of 2 x 201 tokens of hidden 512 27.32 and 26.80.
template <bool FUSED>
__global__ void __launch_bounds__(512) gemm_bf16_rows_small_kernel(GemmDev p) {
  constexpr int STAGES = smem_bytes<64, 64, 8>();
  __shared__ __attribute__((aligned(1024))) unsigned char smem[STAGES + kListBytes<FUSED>];
  lds_idx_t lidx = nullptr;
  const int m = listed_rows<FUSED, STAGES>(p, smem, lidx);
  // (every way out waits for the loads into LDS that are under way)
  if (m > 0 && !few_rows(p, m, smem, lidx)) gemm_tile16<64, 64, 2, 4, 8>(p, m, smem, threadIdx.x, blockIdx.x, lidx);
  wait_vmcnt<0>();
}

template <bool FUSED>
__global__ void __launch_bounds__(512) gemm_bf16_rows_wide_kernel(GemmDev p) {
  // A row list derived from the mask lies behind the stage memory for the whole launch.  (In the stage memory
  // it had to be read before the first load into LDS, a barrier between them, and derived again, seven copies of
  // that code and 152 spilled scalars, in front of every further pass.  Steps, with the shape in line: 2 x 201 tokens
  // of hidden 512 28.5 -> 27.6 us, 1 x 1024 of 4096 with 4 refreshed rows 60.9 -> 60.4, with 205 rows 89.8 -> 89.4.
  // One array for both: see score_proj_kernel.)
  static_assert(kWideSmem + kListBytes<FUSED> <= 160 * 1024, "stage memory and row list must fit the LDS of a CU");
  __shared__ __attribute__((aligned(1024))) unsigned char smem[kWideSmem + kListBytes<FUSED>];
  static_assert(smem_bytes<64, 64, 8>() <= kWideSmem && smem_bytes<128, 48, 5>() <= kWideSmem &&
                    smem_bytes<128, 64, 4>() <= kWideSmem && smem_bytes<128, 96, 4>() <= kWideSmem &&
                    smem_bytes<128, 192, 3>() <= kWideSmem && smem_bytes<128, 128, 4>() <= kWideSmem &&
                    pp_smem_bytes<3>() <= kWideSmem && pp_smem_bytes<4>() <= kWideSmem,
                "shared buffer too small");
  lds_idx_t lidx = nullptr;
  const int m = listed_rows<FUSED, kWideSmem>(p, smem, lidx);
  // (every way out waits for the loads into LDS that are under way)
  if (m <= 0 || few_rows(p, m, smem, lidx)) return wait_vmcnt<0>();
  // Tiles in passes, virtual block id = block id + pass * grid size.  Every thread of the workgroup
  // sees the same m and so takes the same branch and the same number of passes.
  auto passes = [&](int tiles, auto tile) __attribute__((always_inline)) {
    const int per_xcd = (tiles + 7) >> 3;
    for (int vb = blockIdx.x; (vb >> 3) < per_xcd; vb += gridDim.x) {
      if (vb != (int)blockIdx.x) __syncthreads();  // the ring is reused: everybody is done with the last tile
      if (!tile(vb)) break;
    }
    wait_vmcnt<0>();
  };
  const GemmRoute shape = best_tile(m, p.n, true);
  if (shape == GemmRoute::kPp256Cut) {
    // Rounds of 256 x 256 tiles; the tiles of the last round are cut into four 128 x 128 tiles each and
    // spread over all workgroups (one or two short rounds instead of a long, mostly idle one).
    const int G = gridDim.x, tiles_m = (m + 255) / 256, tiles_n = p.n / 256;
    const int total = tiles_m * tiles_n, per_xcd = (total + 7) >> 3, n_vb = per_xcd * 8;  // 8 per XCD slot
    const int whole_end = n_vb - n_vb % G;
    bool first = true;
    auto next_tile = [&]() __attribute__((always_inline)) {
      if (!first) __syncthreads();  // the ring is reused: everybody is done with the last tile
      first = false;
    };
    for (int vb = blockIdx.x; vb < whole_end; vb += G) {
      next_tile();
      gemm_tile_pp<4>(p, m, smem, vb, lidx);
    }
    // child c: the parents of an XCD slot stay on their XCD (c & 7), 4 children per parent
    for (int c = blockIdx.x; c < 4 * (n_vb - whole_end); c += G) {
      const int vb = whole_end + ((c >> 5) << 3) + (c & 7), quarter = (c >> 3) & 3;
      const int unit = (vb & 7) * per_xcd + (vb >> 3);
      if (unit >= total) continue;
      int tm, tn;
      tile_of_unit(unit, tiles_m, tiles_n, tm, tn);
      const int cm = 2 * tm + (quarter >> 1), cn = 2 * tn + (quarter & 1);
      if (cm * 128 >= m) continue;
      next_tile();
      gemm_tile16<128, 128, 2, 4, 4>(p, m, smem, threadIdx.x, 0, lidx, cm, cn);
    }
    return wait_vmcnt<0>();
  }
  switch (shape) {
    case GemmRoute::kPp256:
      return passes(tiles_of(m, p.n, kPpRows, 256), [&](int vb) { return gemm_tile_pp<4>(p, m, smem, vb, lidx); });
    case GemmRoute::kPp192:
      return passes(tiles_of(m, p.n, kPpRows, 192), [&](int vb) { return gemm_tile_pp<3>(p, m, smem, vb, lidx); });
    case GemmRoute::kPp128:
      return passes(tiles_of(m, p.n, kPpRows, 128), [&](int vb) { return gemm_tile_pp<2>(p, m, smem, vb, lidx); });
    case GemmRoute::k128x192:
      return passes(tiles_of(m, p.n, 128, 192), [&](int vb) { return gemm_tile16<128, 192, 2, 4, 3>(p, m, smem, threadIdx.x, vb, lidx); });
    case GemmRoute::k128x128:
      return passes(tiles_of(m, p.n, 128, 128), [&](int vb) { return gemm_tile16<128, 128, 2, 4, 4>(p, m, smem, threadIdx.x, vb, lidx); });
    case GemmRoute::k128x96:
      return passes(tiles_of(m, p.n, 128, 96), [&](int vb) { return gemm_tile16<128, 96, 4, 2, 4>(p, m, smem, threadIdx.x, vb, lidx); });
    case GemmRoute::k128x64:
      return passes(tiles_of(m, p.n, 128, 64), [&](int vb) { return gemm_tile16<128, 64, 4, 2, 4>(p, m, smem, threadIdx.x, vb, lidx); });
    case GemmRoute::k128x48:
      return passes(tiles_of(m, p.n, 128, 48), [&](int vb) { return gemm_tile16<128, 48, 8, 1, 5>(p, m, smem, threadIdx.x, vb, lidx); });
    default:
      return passes(tiles_of(m, p.n, 64, 64), [&](int vb) { return gemm_tile16<64, 64, 2, 4, 8>(p, m, smem, threadIdx.x, vb, lidx); });
  }
}

// ---- scored query columns of all rows, with the score ---------------------------------
// One launch for what were three dependent steps of a few microseconds each (projection in
// k-range slabs, a second kernel that added the slabs and scored): BM rows x all WIDTH scored
// columns per workgroup, so that a workgroup holds whole queries and can score them.  What bounds
// it is the operands that a CU pulls, (BM + WIDTH) rows of k; with few row tiles k is cut over
// KP workgroups, each of which leaves its sums at device scope (as in gemm_tile_pp), and the
// last one to arrive adds them up.
// Sum over k: that of the caller's ranges of k, added up as a binary tree whatever BM and KP are,
// so the route (workspace or not) does not show in a query.
// Measured (projection + score + the gap between them -> this launch, inside a step): 1024 rows
// 7.6 + 4.9 + 2.4 -> 11 us, 8192 rows 45 + 7.7 + 2.4 -> 38 us, 16384 rows 52 + 9.4 + 2.4 -> 45 us.
struct ScoreProjDev {
  const bf16_t* a;
  const bf16_t* wt;
  const int32_t* idx;
  float* q_prev;
  float* scores;
  uint8_t* mask;
  float* sums;
  unsigned* count;
  int k, m, k_parts, ranges;  // workgroups per row tile; ranges of the summation tree
  int force_refresh, batch, seq, prefix;
  float threshold;
};

template <int BM, int WIDTH, int WAVES_M, int WAVES_N>
__global__ void __launch_bounds__(WAVES_M* WAVES_N * 64) score_proj_kernel(ScoreProjDev p) {
  constexpr int NW = WAVES_M * WAVES_N, NT = NW * 64, STAGES = 5;
  constexpr int WM = BM / WAVES_M, WN = WIDTH / WAVES_N;
  constexpr int TM = WM / 16, TN = WN / 16, KS = BK / 32;
  constexpr int STAGE_BYTES = (BM + WIDTH) * ROW_BYTES;
  constexpr int GROUPS = (BM + WIDTH) / 8;
  constexpr int LPW = (GROUPS + NW - 1) / NW;  // surplus loads repeat the last group
  constexpr int LDQ = score_query_stride(WIDTH);
  static_assert(WM % 16 == 0 && WN % 16 == 0 && BM % NW == 0, "wave tiles of 16 x 16, whole rows per wave");
  static_assert(LPW * (STAGES - 1) < 64, "vmcnt range");
  // (one LDS array only: with a second one the compiler tracks which of them a global -> LDS load
  // may write, and puts s_waitcnt vmcnt(0) in front of the fragment reads, which drains the ring)
  __shared__ __attribute__((aligned(1024))) unsigned char smem[STAGES * STAGE_BYTES];
  // whether this workgroup is the last one lies behind the queries, which a wave may write while another
  // one still reads it
  constexpr int ARRIVED = score_arrived_offset(BM, WIDTH);
  static_assert(ARRIVED + 4 <= STAGES * STAGE_BYTES, "the flag must fit into the stage memory");
  int& last_here = *reinterpret_cast<int*>(smem + ARRIVED);

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // frozen tokens: always reused, never scored
  for (long i = (long)blockIdx.x * NT + tid; i < (long)p.batch * p.prefix; i += (long)gridDim.x * NT) {
    const long tok = i / p.prefix * p.seq + i % p.prefix;
    if (p.scores) p.scores[tok] = 0.f;
    p.mask[tok] = 1;
  }

  const int tile = blockIdx.x / p.k_parts, part = blockIdx.x % p.k_parts;
  const int m0 = tile * BM;
  const int wave_m = wave % WAVES_M, wave_n = wave / WAVES_M;
  const int l16 = lane & 15, kq = lane >> 4;
  const int KT = p.k / BK / p.k_parts;      // k-steps of this workgroup
  const int range = p.k / BK / p.ranges;    // k-steps of a range of the tree

  const bf16_t* src[LPW];
  int grp[LPW];
#pragma unroll
  for (int i = 0; i < LPW; ++i) {
    grp[i] = wave * LPW + i < GROUPS ? wave * LPW + i : GROUPS - 1;
    const int r = grp[i] * 8 + (lane >> 3);
    const long off = (long)part * KT * BK + ((lane & 7) ^ ((r >> 1) & 7)) * 8;
    if (r < BM) {
      const int row = m0 + r < p.m ? m0 + r : p.m - 1;
      src[i] = p.a + (long)(p.idx ? p.idx[row] : row) * p.k + off;
    } else {
      src[i] = p.wt + (long)(r - BM) * p.k + off;
    }
  }
  auto issue_loads = [&](int kt) __attribute__((always_inline)) {
    unsigned char* base = smem + (kt % STAGES) * STAGE_BYTES;
    const int k = kt < KT ? kt : KT - 1;
#pragma unroll
    for (int i = 0; i < LPW; ++i)
      __builtin_amdgcn_global_load_lds((gptr_t)(src[i] + k * BK), (lptr_t)(base + grp[i] * 8 * ROW_BYTES), 16, 0, 0);
  };

  f32x4 acc[TM][TN], level[3][TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = level[0][i][j] = level[1][i][j] = level[2][i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int sw = (l16 >> 1) & 7;
  const int a_row_off = (wave_m * WM + l16) * ROW_BYTES;
  const int b_row_off = (BM + wave_n * WN + l16) * ROW_BYTES;

#pragma unroll
  for (int s = 0; s < STAGES - 1; ++s) issue_loads(s);
  int done = 0, in_range = 0;  // ranges complete, k-steps of the current one
  for (int kt = 0; kt < KT; ++kt) {
    wait_vmcnt_and_barrier<LPW*(STAGES - 2)>();
    issue_loads(kt + STAGES - 1);
    const unsigned char* st = smem + (kt % STAGES) * STAGE_BYTES;
    bf16x8 fa[KS][TM], fb[KS][TN];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const int koff = ((ks * 4 + kq) ^ sw) * 16;
#pragma unroll
      for (int i = 0; i < TM; ++i) fa[ks][i] = *reinterpret_cast<const bf16x8*>(st + a_row_off + i * 16 * ROW_BYTES + koff);
#pragma unroll
      for (int j = 0; j < TN; ++j) fb[ks][j] = *reinterpret_cast<const bf16x8*>(st + b_row_off + j * 16 * ROW_BYTES + koff);
    }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[ks][j], fa[ks][i], acc[i][j], 0, 0, 0);
    if (++in_range < range) continue;
    // a range is complete: up the tree (the last one of the workgroup ends as its whole sum in acc)
    in_range = 0;
    const bool last = kt + 1 == KT;
    bool carry = true;
#pragma unroll
    for (int l = 0; l < 3; ++l) {
      if (!carry) break;
      if ((done >> l) & 1) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j) acc[i][j] = level[l][i][j] + acc[i][j];
      } else if (!last) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j) {
            level[l][i][j] = acc[i][j];
            acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
          }
        carry = false;
      }
    }
    ++done;
  }
  wait_vmcnt<0>();
  __syncthreads();

  if (p.k_parts > 1) {
    constexpr int kDeviceScope = 16;  // cache policy sc1
    constexpr int kSlot = BM * WIDTH * 4;
    const auto slots = __builtin_amdgcn_make_buffer_rsrc(p.sums + (long)tile * p.k_parts * (BM * WIDTH), 0, p.k_parts * kSlot, 0x00027000);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, acc[i][j]), slots, part * kSlot + ((i * TN + j) * NT + tid) * 16, 0, kDeviceScope);
    wait_vmcnt<0>();
    __syncthreads();
    if (tid == 0) last_here = arrive_last(p.count + tile, p.k_parts);
    __syncthreads();
    if (!last_here) return;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        f32x4 w[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          w[q] = f32x4{0.f, 0.f, 0.f, 0.f};
          if (q < p.k_parts)
            w[q] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(slots, q * kSlot + ((i * TN + j) * NT + tid) * 16, 0, kDeviceScope));
        }
        f32x4 v = w[0] + w[1];  // (the tree above the workgroups)
        if (p.k_parts > 2) v += w[2] + w[3];
        if (p.k_parts > 4) v += (w[4] + w[5]) + (w[6] + w[7]);
        acc[i][j] = v;
      }
  }

  // acc[i][j][e] = query[row, col]: row = wave_m*WM + 16 i + l16, col = wave_n*WN + 16 j + 4 kq + e
  float* qs = reinterpret_cast<float*>(smem);
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
      *reinterpret_cast<f32x4*>(qs + (wave_m * WM + i * 16 + l16) * LDQ + wave_n * WN + j * 16 + kq * 4) = acc[i][j];
  __syncthreads();
  // score: a wave per row, two neighbouring channels per lane, the three sums with one lane
  // assignment and one butterfly (an unchanged query gives dot == |q|^2 == |p|^2 bit for bit)
  constexpr int RPW = BM / NW;
  const int c = lane * 2;
  f32x2 prev[RPW];
  long tok[RPW];
#pragma unroll
  for (int r = 0; r < RPW; ++r) {
    const int row = m0 + wave * RPW + r;
    const int listed = row < p.m ? row : p.m - 1;
    tok[r] = p.idx ? p.idx[listed] : listed;
    prev[r] = c < WIDTH ? *reinterpret_cast<const f32x2*>(p.q_prev + tok[r] * WIDTH + c) : f32x2{0.f, 0.f};
  }
#pragma unroll
  for (int r = 0; r < RPW; ++r) {
    if (m0 + wave * RPW + r >= p.m) break;
    f32x2 q = {0.f, 0.f};
    if (c < WIDTH) {
      q = *reinterpret_cast<const f32x2*>(qs + (wave * RPW + r) * LDQ + c);
      *reinterpret_cast<f32x2*>(p.q_prev + tok[r] * WIDTH + c) = q;  // the score cache takes this step's query
    }
    const float dot = wave_sum(fmaf(q[1], prev[r][1], q[0] * prev[r][0]));
    const float nq = wave_sum(fmaf(q[1], q[1], q[0] * q[0]));
    const float np = wave_sum(fmaf(prev[r][1], prev[r][1], prev[r][0] * prev[r][0]));
    if (lane == 0) {
      const float s = drift_score(dot, nq, np);
      if (p.scores) p.scores[tok[r]] = s;
      p.mask[tok[r]] = (!p.force_refresh && s <= p.threshold) ? 1 : 0;
    }
  }
}

GemmDev to_dev(const GemmArgs& g) {
  GemmDev p;
  p.a = static_cast<const bf16_t*>(g.a);
  p.wt = static_cast<const bf16_t*>(g.wt);
  p.idx = g.idx;
  p.m_dev = g.m_dev;
  p.c0 = static_cast<bf16_t*>(g.c[0]);
  p.c1 = static_cast<bf16_t*>(g.c[1]);
  p.c2 = static_cast<bf16_t*>(g.c[2]);
  p.c32 = g.c32;
  p.lda = g.lda;
  p.n = g.n;
  p.k = g.k;
  p.m_max = g.m_max;
  p.ldc = g.ldc;
  p.seg_n = g.seg_n;
  p.c32_cols = g.c32_cols;
  p.k_parts = 1;
  p.c32_part_stride = 0;
  p.rope = g.rope;
  p.rope_cols = g.rope_cols;
  p.rope_dh = g.rope_dh;
  p.rope_seq = g.rope_seq;
  p.swiglu_pairs = g.swiglu_pairs;
  p.sel_mask = g.sel_mask;
  p.sel_batch = g.sel_batch;
  p.sel_seq = g.sel_seq;
  p.sel_idx_out = g.sel_idx_out;
  p.sel_idx_out2 = g.sel_idx_out2;
  p.sel_off_out = g.sel_off_out;
  p.sel_count_out = g.sel_count_out;
  p.ahead = 0;
  p.split_tiles = g.split_tiles;
  p.split_count = g.split_count;
  p.part_n = g.part_n;
  p.part_idx = g.part_idx;
  p.part_m_dev = g.part_m_dev;
  return p;
}

int grid_for(int tiles) { return ((tiles + 7) / 8) * 8; }

// Outputs larger than half of the last-level cache (256 MB) are stored past the L2: what the stages behind them read first is
// no longer there anyway, and the operands stay in its place (us, stored through the L2 and past it, in a step of 8 x 2048 tokens of hidden 4096:
// Q, K and V, 403 MB, 1136 and 1130, the score, the normalisation and the residual sum around them 10.4 and 9.0, 46.2 and 45.7, 70.0
// and 64.9).  Smaller ones are not: 25 MB, 1 x 1024 x 12288, leave the attention behind them 32.2 us, and 33.4 stored past it.
constexpr long kStreamBytes = 128l << 20;
template <int TN>
hipError_t launch_quad(const GemmArgs& g, hipStream_t s) {
  const int tiles = grid_for(tiles_of(g.m_max, g.n, kPpRows, 64 * TN));
  const dim3 grid(tiles < kWideGrid ? tiles : kWideGrid);
  if (TN == 4 && (long)g.m_max * g.n * (g.swiglu_pairs ? 1 : 2) > kStreamBytes)
    hipLaunchKernelGGL((gemm_bf16_quad_kernel<TN, TN == 4>), grid, dim3(256), 0, s, to_dev(g));
  else
    hipLaunchKernelGGL((gemm_bf16_quad_kernel<TN, false>), grid, dim3(256), 0, s, to_dev(g));
  return hipGetLastError();
}

template <int BM, int BN, int WAVES_M, int WAVES_N, int STAGES>
hipError_t launch_ranges(const GemmArgs& g, hipStream_t s) {
  GemmDev p = to_dev(g);
  p.k_parts = g.k_parts;
  p.c32_part_stride = g.c32_part_stride;
  hipLaunchKernelGGL((gemm_bf16_ranges_kernel<BM, BN, WAVES_M, WAVES_N, STAGES>),
                     dim3(grid_for(tiles_of(g.m_max, g.n, BM, BN) * p.k_parts)), dim3(WAVES_M * WAVES_N * 64), 0, s, p);
  return hipGetLastError();
}

template <int BM, int BN, int WAVES_M, int WAVES_N, int STAGES>
hipError_t launch_tile16(const GemmArgs& g, hipStream_t s) {
  hipLaunchKernelGGL((gemm_bf16_tile16_kernel<BM, BN, WAVES_M, WAVES_N, STAGES>),
                     dim3(grid_for(tiles_of(g.m_max, g.n, BM, BN))), dim3(512), 0, s, to_dev(g));
  return hipGetLastError();
}

template <int TN, bool SPLIT = false>
hipError_t launch_pp(const GemmArgs& g, hipStream_t s) {
  const int tiles = tiles_of(g.m_max, g.n, kPpRows, 64 * TN);
  if (SPLIT && (tiles > kSplitTiles || !g.split_tiles || !g.split_count)) return hipErrorInvalidValue;
  hipLaunchKernelGGL((gemm_bf16_pp_kernel<TN, SPLIT>), dim3(grid_for(SPLIT ? 2 * tiles : tiles)), dim3(512), 0, s,
                     to_dev(g));
  return hipGetLastError();
}

hipError_t launch_rows_wide(const GemmArgs& g, hipStream_t s) {
  // as many as the smallest tiles, or the column groups of the stream over the weights, whichever are more
  const int small = tiles_of(g.m_max, g.n, 64, 64), groups = g.m_max > 0 ? g.n / 16 : 0;
  int blocks = small > groups ? small : groups;
  if (blocks == 0) return hipSuccess;
  if (blocks > kWideGrid) blocks = kWideGrid;
  blocks = grid_for(blocks);
  GemmDev p = to_dev(g);
  p.ahead = ahead_loads(g.n, blocks);
  if (small <= kWideGrid && g.sel_mask)
    hipLaunchKernelGGL(gemm_bf16_rows_small_kernel<true>, dim3(blocks), dim3(512), 0, s, p);
  else if (small <= kWideGrid)
    hipLaunchKernelGGL(gemm_bf16_rows_small_kernel<false>, dim3(blocks), dim3(512), 0, s, p);
  else if (g.sel_mask)
    hipLaunchKernelGGL(gemm_bf16_rows_wide_kernel<true>, dim3(blocks), dim3(512), 0, s, p);
  else
    hipLaunchKernelGGL(gemm_bf16_rows_wide_kernel<false>, dim3(blocks), dim3(512), 0, s, p);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_gemm_bf16(const GemmArgs& g, hipStream_t s) {
  if (g.part_n > 0) {
    if (g.m_max == 0) return hipSuccess;
    if (g.m_dev || g.sel_mask || g.c32 || g.swiglu_pairs || !g.part_idx || !g.part_m_dev || g.part_n >= g.n || g.part_n % 64 != 0 ||
        g.k < kQuadMinSteps * BK)
      return hipErrorInvalidValue;
    hipLaunchKernelGGL(gemm_bf16_part_kernel, dim3(kWideGrid), dim3(256), 0, s, to_dev(g));
    return hipGetLastError();
  }
  if (g.m_dev || g.sel_mask) return launch_rows_wide(g, s);
  if (g.m_max == 0) return hipSuccess;
  switch (gemm_route(g.m_max, g.n, g.k, g.k_parts, g.split_tiles && !g.c32)) {
    case GemmRoute::kPp128Split: return launch_pp<2, true>(g, s);
    case GemmRoute::kQuad256: return launch_quad<4>(g, s);
    case GemmRoute::kQuad192: return launch_quad<3>(g, s);
    case GemmRoute::kPp256: return launch_pp<4>(g, s);
    case GemmRoute::kPp192: return launch_pp<3>(g, s);
    case GemmRoute::kPp128: return launch_pp<2>(g, s);
    case GemmRoute::k128x192: return launch_tile16<128, 192, 2, 4, 3>(g, s);
    case GemmRoute::k128x128: return launch_tile16<128, 128, 2, 4, 4>(g, s);
    case GemmRoute::k128x96: return launch_tile16<128, 96, 4, 2, 4>(g, s);
    case GemmRoute::k64x128: return launch_tile16<64, 128, 2, 4, 5>(g, s);
    case GemmRoute::k64x96: return launch_tile16<64, 96, 4, 2, 6>(g, s);
    case GemmRoute::k64x64: return launch_tile16<64, 64, 2, 4, 8>(g, s);
    case GemmRoute::kTile128: return launch_ranges<128, 128, 4, 2, 4>(g, s);
    case GemmRoute::kTile64: return launch_ranges<64, 64, 2, 2, 4>(g, s);
    case GemmRoute::k128x48: case GemmRoute::k128x64: case GemmRoute::kPp256Cut: break;  // (listed rows)
  }
  return hipErrorInvalidValue;
}

hipError_t launch_score_proj(const ScoreProjArgs& g, hipStream_t s) {
  if (g.m == 0) return hipSuccess;
  const int ranges = g.k_ranges;
  // Rows per workgroup and workgroups per row tile, by what a workgroup takes (us): its operands at
  // 100 KB/us; when k is cut, 3 for the hand-over and the slots that the last workgroup reads back at
  // 40 KB/us; 0.04 per row to score.  Fitted at 1024 rows of 4096, width 128 (rows / workgroups per
  // tile): 16/4 11.0 us, 16/2 13.6, 32/4 12.7, 32/8 13.1, 64/4 16.1, 64/8 16.4.
  int bm = 64, kp = 1;
  double best = 1e30;
  for (int b = 16; b <= 64; b *= 2)
    for (int q = 1; q <= ranges; q *= 2) {
      const long tiles = (g.m + b - 1) / b;
      const size_t slots = (size_t)tiles * q * b * g.width;
      if (q > 1 && (!g.sums || tiles > kScoreTiles || slots > g.sums_elems)) continue;
      const double rounds = (double)((tiles * q + 255) / 256);
      const double pull = rounds * (b + g.width) * (double)(g.k / q) * 2 / 100e3;
      const double cost = pull + (q > 1 ? 3.0 + (double)q * b * g.width * 4 / 40e3 : 0.0) + 0.04 * b;
      if (cost < best) {
        best = cost;
        bm = b;
        kp = q;
      }
    }
  ScoreProjDev p;
  p.a = static_cast<const bf16_t*>(g.a);
  p.wt = static_cast<const bf16_t*>(g.wt);
  p.idx = g.idx;
  p.q_prev = g.q_prev;
  p.scores = g.scores;
  p.mask = g.mask;
  p.sums = g.sums;
  p.count = g.count;
  p.k = g.k;
  p.m = g.m;
  p.k_parts = kp;
  p.ranges = ranges;
  p.force_refresh = g.force_refresh;
  p.batch = g.batch;
  p.seq = g.seq;
  p.prefix = g.prefix;
  p.threshold = g.threshold;
  const dim3 grid((unsigned)((g.m + bm - 1) / bm * kp));
  if (g.width == 128) {
    if (bm == 16) hipLaunchKernelGGL((score_proj_kernel<16, 128, 1, 8>), grid, dim3(512), 0, s, p);
    else if (bm == 32) hipLaunchKernelGGL((score_proj_kernel<32, 128, 2, 4>), grid, dim3(512), 0, s, p);
    else hipLaunchKernelGGL((score_proj_kernel<64, 128, 2, 4>), grid, dim3(512), 0, s, p);
  } else if (g.width == 64) {
    if (bm == 16) hipLaunchKernelGGL((score_proj_kernel<16, 64, 1, 4>), grid, dim3(256), 0, s, p);
    else if (bm == 32) hipLaunchKernelGGL((score_proj_kernel<32, 64, 2, 4>), grid, dim3(512), 0, s, p);
    else hipLaunchKernelGGL((score_proj_kernel<64, 64, 4, 2>), grid, dim3(512), 0, s, p);
  } else {
    return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace dare
