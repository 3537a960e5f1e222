// Bidirectional multi-head attention for a selected set of query rows on the
// gfx950 matrix cores (App. E.2; Alg. 1 line 10; Alg. 2 line 8):
//     out[t, h] = softmax(q[t, h] . K_b[:, h]^T / sqrt(Dh)) V_b[:, h]
// with t running over all tokens or over the refreshed tokens of each sequence.
//
// A workgroup serves 32 * QW query rows of one (sequence, head) with QW * KW waves:
// wave (qw, kw) owns 32 query rows and every KW-th tile of TK keys.  K and V tiles go
// from global memory straight into LDS (global_load_lds_dwordx4) through a ring of
// NST stages, rows kept as they are in memory ([key][channel]); bank conflicts are
// removed by fetching, into the LDS slot a lane owns, the 16-byte chunk that an XOR
// of the key index assigns to it.
//
// Each wave computes the TRANSPOSED logits S^T = K Q^T with
// v_mfma_f32_32x32x16_bf16, so a lane holds the logits of ONE query row: the running
// max / sum of the online softmax are per-lane scalars (one exchange with lane^32),
// and the probabilities are already in the register layout of the second operand of
// O^T = V^T P^T.  The first operand, V^T, is read from the row-major V tile with the
// LDS transpose read ds_read_b64_tr_b16 (a lane receives 4 consecutive keys of one
// channel), so V needs no transposition pass.
//
// With KW > 1 the key-waves of a query block each keep their own running
// (max, sum, O) and are merged once at the end through LDS, in a fixed order.
// Few query rows (the refreshed rows of a step) use narrow query blocks with KW > 1,
// which turns the available waves towards the key axis and fills the chip, and with very few
// of them the keys of a block are cut over workgroups as well; many rows use wide blocks (128
// rows with two key-waves, or without any when there are enough of them; 256 rows with heads of 64 channels), which
// re-read K and V less often.  attn_route.h holds the rule.
// Blocks of 128 rows of heads of 128 channels run attn_wide, which takes 16 x 16 x 32 MFMAs and lets softmax and products of
// neighbouring key subtiles overlap; everything else runs attn_block, described here.
#include <type_traits>

#include "dare_common.h"

namespace dare {
namespace {

constexpr float kLog2e = 1.4426950408889634f;

struct AttnDev {
  const bf16_t* q;
  const bf16_t* k;
  const bf16_t* v;
  bf16_t* out;
  const int32_t* idx;
  const int32_t* sel_off;
  int seq, d;
  int n_heads, n_pairs, n_qt;  // heads, batch*heads, query blocks launched per (sequence, head)
  int batch;
  int turn, at_once;           // order of the workgroups, readers ahead (attn_turn, attn_at_once)
  // attn_wide without key-waves (attn_second_reference): tile to whose maximum the reference exponent moves (0: none), sum of a
  // lane's probabilities from which on maxima are looked for, and how far above it in base 2 one has to be
  int second;
  float limit, grow;
  // keys of a query block cut over workgroups (attn_rows_bf16_kernel): partial results, and
  // counters that are 0 before and after the launch; nullptr = never cut
  float* part_out;
  unsigned* part_count;
  float scale_log2;
};

typedef __attribute__((address_space(3))) void* lptr_t;
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4* lds_s16x4_ptr;

template <int N>
__device__ __forceinline__ void wait_vmcnt_and_barrier() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}
__device__ __forceinline__ void wait_all_and_barrier() {
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// 16 bytes per lane from global memory to LDS address lds + 16 lane, waited for by hand.  Not the
// builtin: the compiler would put s_waitcnt vmcnt(0) in front of the first transpose read of every
// step (it cannot tell that such a read and a load into another stage do not meet), which drains
// the ring and leaves no stage in flight under the value product.
__device__ __forceinline__ void load_to_lds(const bf16_t* src, unsigned char* lds) {
  // (the address is an operand in M0, set by the compiler, which then knows what M0 holds; a wait state
  // between the move to M0 and the load)
  asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(src), "{m0}"((unsigned)(size_t)(lptr_t)lds) : "memory");
}

template <int DH, int KW, int TK, int NST>
constexpr int attn_smem_bytes() {
  return NST * KW * 2 * TK * DH * 2;
}

// XOR applied to the 16-byte chunk index of a K row / V row (see the header).
template <int DH>
__device__ __forceinline__ int k_swizzle(int key) {
  return DH == 128 ? (key & 15) : ((key >> 1) & 7);
}
template <int DH>
__device__ __forceinline__ int v_swizzle(int key) {
  return DH == 128 ? ((key & 3) << 2) : (((key >> 1) & 1) << 2);
}

// One query block.  b, h: sequence and head; qt: query block index inside the row set
// [off, off + cnt) of the sequence.  Called by all QW*KW waves of the workgroup.
template <int DH, int QW, int KW, int TK, int NST>
__device__ __forceinline__ void attn_block(const AttnDev& p, int b, int h, int qt, int cnt, int off,
                                           unsigned char* smem, const int tid, int part = 0, int n_parts = 1,
                                           int block = 0) {
  constexpr int NW = QW * KW;
  constexpr int ROWB = DH * 2;             // bytes per K or V row of one head
  constexpr int CPR = DH / 8;              // 16-byte chunks per row
  constexpr int RPL = 64 / CPR;            // rows covered by one wave load
  constexpr int TILE_BYTES = TK * ROWB;
  constexpr int STAGE_BYTES = KW * 2 * TILE_BYTES;
  constexpr int NL = STAGE_BYTES / 1024;   // wave loads per stage
  constexpr int LPW = NL / NW;
  constexpr int KSTEPS = DH / 16;          // k-steps of the logits product
  constexpr int OT = DH / 32;              // 32-channel tiles of the output
  constexpr int ST = TK / 32;              // 32-key tiles of the logits
  constexpr int PS = TK / 16;              // 16-key slices of the value product
  static_assert(NL % NW == 0, "stage loads must divide among the waves");
  static_assert(LPW * (NST - 1) < 64, "vmcnt range");

  const int T = p.seq;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // (a scalar: M0 addressing)
  // (the key-waves of few query rows on a SIMD each: where the second half of a block holds no rows, the
  // first one has every SIMD's matrix core to itself)
  const int qw = KW == 4 ? (unsigned)wave / KW : (unsigned)wave % QW, kw = KW == 4 ? (unsigned)wave % KW : (unsigned)wave / QW;
  const int l32 = lane & 31, half = lane >> 5;

  // the query row of this lane
  const int j = qt * (32 * QW) + qw * 32 + l32;
  const bool valid = j < cnt;
  const bool any_row = qt * (32 * QW) + qw * 32 < cnt;  // (the same in all lanes: a wave without rows only loads)
  const int jc = valid ? j : cnt - 1;
  int tok = p.idx ? p.idx[off + jc] : off + jc;

  bf16x8 qf[KSTEPS];
  {
    const bf16_t* qrow = p.q + (long)tok * p.d + h * DH + half * 8;
#pragma unroll
    for (int ks = 0; ks < KSTEPS; ++ks)
      qf[ks] = *reinterpret_cast<const bf16x8*>(qrow + ks * 16);
  }

  // ---- global -> LDS: stage rows are, per key-wave tile, TK rows of K then TK of V ----
  const bf16_t* kbase = p.k + (long)b * T * p.d + h * DH;
  const bf16_t* vbase = p.v + (long)b * T * p.d + h * DH;
  int ld_key[LPW];           // key of this lane's row at step 0
  const bf16_t* ld_src[LPW]; // K or V base + chunk offset
#pragma unroll
  for (int i = 0; i < LPW; ++i) {
    // (unsigned: the compiler knows no range of a wave number read from one lane, and signed quotients
    // took 80 instructions in front of the first load)
    const unsigned sr = (unsigned)(wave * LPW + i) * RPL + (unsigned)lane / CPR;  // row within the stage
    const int tile = sr / (2 * TK), within = sr % (2 * TK);
    const bool is_v = within >= TK;
    const int key_local = (unsigned)within % TK;
    const int chunk = ((unsigned)lane % CPR) ^ (is_v ? v_swizzle<DH>(key_local) : k_swizzle<DH>(key_local));
    ld_key[i] = tile * TK + key_local;
    ld_src[i] = (is_v ? vbase : kbase) + chunk * 8;
  }
  auto issue_loads = [&](int step, int buf) __attribute__((always_inline)) {
    unsigned char* base = smem + buf * STAGE_BYTES + wave * LPW * 1024;
#pragma unroll
    for (int i = 0; i < LPW; ++i) {
      int key = ld_key[i] + step * (KW * TK);
      key = key < T ? key : T - 1;
      load_to_lds(ld_src[i] + (long)key * p.d, base + i * 1024);
    }
  };

  // ---- per-lane LDS read offsets ----
  // K fragment: row (32 kt + l32), chunk (2 ks + half) ^ k_swizzle(row)
  int k_off[KSTEPS];
#pragma unroll
  for (int ks = 0; ks < KSTEPS; ++ks)
    k_off[ks] = l32 * ROWB + (((ks * 2 + half) ^ k_swizzle<DH>(l32)) * 16);
  // V^T fragment by transpose read: within each group of 16 lanes, lane r supplies the
  // address of key (r >> 2) of the 4-key run, channels 4 (r & 3) .. +3 of the 16
  // channels the group covers; lane i of the group receives those 4 keys at channel i.
  int v_off[OT];
  {
    const int r = lane & 15, e = r >> 2, jj = r & 3;
    const int key_l = half * 4 + e;                       // + 16 s4 + 8 which
    const int c_lane = 2 * ((lane >> 4) & 1) + (jj >> 1); // chunk within the 32-channel tile
    const int vs = v_swizzle<DH>(key_l) >> 2;
#pragma unroll
    for (int t = 0; t < OT; ++t)
      v_off[t] = key_l * ROWB + (((t ^ vs) * 4 + c_lane) * 16) + (jj & 1) * 8;
  }

  f32x16 acc_o[OT];
#pragma unroll
  for (int t = 0; t < OT; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc_o[t][r] = 0.f;
  float m_run = -INFINITY, l_run = 0.f;

  auto compute = [&](int buf, int kv0) __attribute__((always_inline)) {
    const unsigned char* kb = smem + buf * STAGE_BYTES + kw * 2 * TILE_BYTES;
    const unsigned char* vb = kb + TILE_BYTES;
    // S^T tile: TK keys x 32 query rows
    f32x16 acc_s[ST];
#pragma unroll
    for (int kt = 0; kt < ST; ++kt) {
#pragma unroll
      for (int r = 0; r < 16; ++r) acc_s[kt][r] = 0.f;
#pragma unroll
      for (int ks = 0; ks < KSTEPS; ++ks) {
        const bf16x8 kf = *reinterpret_cast<const bf16x8*>(kb + kt * 32 * ROWB + k_off[ks]);
        acc_s[kt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[ks], acc_s[kt], 0, 0, 0);
      }
    }
    // register r of tile kt is key kv0 + kt*32 + (r/4)*8 + half*4 + r%4
    if (kv0 + TK > T) {  // last, ragged tile only (uniform branch): keys past the end
#pragma unroll
      for (int kt = 0; kt < ST; ++kt)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int key = kv0 + kt * 32 + (r >> 2) * 8 + half * 4 + (r & 3);
          if (key >= T) acc_s[kt][r] = -INFINITY;
        }
    }
    float m_tile = -INFINITY;
#pragma unroll
    for (int kt = 0; kt < ST; ++kt)
#pragma unroll
      for (int r = 0; r < 16; ++r) m_tile = fmaxf(m_tile, acc_s[kt][r]);
    m_tile = fmaxf(m_tile, __shfl_xor(m_tile, 32, 64)) * p.scale_log2;  // scale > 0
    // Lazy rescaling: the reference exponent m_run of a row only moves when the row's
    // maximum has grown by more than 2^8 over it, so probabilities stay below 256 and
    // the accumulator rescale (a pass over all of O) is skipped for almost every tile.
    // The result does not depend on the reference: O and the row sum share it.
    const bool grow = m_tile > m_run + 8.0f;
    if (__any(grow)) {
      const float m_new = grow ? m_tile : m_run;
      const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
      m_run = m_new;
      l_run *= alpha;
#pragma unroll
      for (int t = 0; t < OT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc_o[t][r] *= alpha;
    }
    const float neg_m = -m_run;
    const bf16x2 ones = {(bf16_t)1.0f, (bf16_t)1.0f};
    float l_tile = 0.f;
    bf16x8 pf[PS];
#pragma unroll
    for (int kt = 0; kt < ST; ++kt)
#pragma unroll
      for (int r = 0; r < 16; r += 2) {
        f32x2 pr;
        pr[0] = __builtin_amdgcn_exp2f(fmaf(acc_s[kt][r], p.scale_log2, neg_m));
        pr[1] = __builtin_amdgcn_exp2f(fmaf(acc_s[kt][r + 1], p.scale_log2, neg_m));
        const bf16x2 pb = __builtin_convertvector(pr, bf16x2);
        // the row sum is taken over the probabilities as rounded for the value product,
        // so numerator and denominator carry the same rounding (v_dot2: += pb[0] + pb[1])
        l_tile = __builtin_amdgcn_fdot2_f32_bf16(pb, ones, l_tile, false);
        pf[kt * 2 + (r >> 3)][r & 7] = pb[0];
        pf[kt * 2 + (r >> 3)][(r & 7) + 1] = pb[1];
      }
    l_run += l_tile;

    // O^T += V^T P^T.  Slot s of P slice s4 is key 16 s4 + 8 (s/4) + 4 half + s%4.
#pragma unroll
    for (int t = 0; t < OT; ++t) {
#pragma unroll
      for (int s4 = 0; s4 < PS; ++s4) {
        const unsigned char* va = vb + s4 * 16 * ROWB + v_off[t];
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(va));
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(va + 8 * ROWB));
        const bf16x4 blo = __builtin_bit_cast(bf16x4, lo), bhi = __builtin_bit_cast(bf16x4, hi);
        const bf16x8 vf = __builtin_shufflevector(blo, bhi, 0, 1, 2, 3, 4, 5, 6, 7);
        acc_o[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pf[s4], acc_o[t], 0, 0, 0);
      }
    }
  };

  // ---- pipeline over the key tiles ----
  const int n_tiles = (T + TK - 1) / TK;
  const int all_steps = (n_tiles + KW - 1) / KW;
  const int first = all_steps * part / n_parts, n_steps = all_steps * (part + 1) / n_parts - first;
#pragma unroll
  for (int s = 0; s < NST - 1; ++s) issue_loads(first + (s < n_steps ? s : n_steps - 1), s);
  // (the queries in registers before the loop, or the compiler waits for them in every step)
#pragma unroll
  for (int ks = 0; ks < KSTEPS; ++ks) asm volatile("" : "+v"(qf[ks]));
  for (int step = 0; step < n_steps; ++step) {
    // step's tiles have landed for every wave, and everybody is done with step-1's
    wait_vmcnt_and_barrier<LPW*(NST - 2)>();
    const int nxt = step + NST - 1;
    // (past the end a ring of more than two stages loads the last step again, to keep the count of loads
    // in flight; with two stages every wait is for all of them, and a block of one step ends without waiting
    // for a load that nobody reads: 2048 x 8 tokens of 16 heads 236 -> 220 us, 16 x 256 of 32 heads 43 -> 36)
    if (NST > 2 || nxt < n_steps) issue_loads(first + (nxt < n_steps ? nxt : n_steps - 1), nxt % NST);
    const int tile = (first + step) * KW + kw;
    if (tile < n_tiles && any_row) compute(step % NST, tile * TK);
  }
  float l_all = l_run + __shfl_xor(l_run, 32, 64);

  // ---- merge the key-waves (fixed order), normalise, store ----
  // Every key-wave merges, and stores, its share of the channels: OWN of the accumulator registers of a
  // lane.  (One wave merging all of them took 2.7 us of the 16 us of a launch over 1024 keys.)
  constexpr int REGS = OT * 16, OWN = REGS / KW;
  f32x4 own[OWN / 4];  // registers kw OWN .. of the merged accumulator
  if constexpr (KW > 1) {
    constexpr int ML = QW * KW * (KW - 1) * OWN * 64;  // (max, sum) of every wave behind the registers
    static_assert((ML + QW * KW * 64 * 2) * 4 <= attn_smem_bytes<DH, KW, TK, NST>(),
                  "the merge area must fit into the stage memory");
    wait_all_and_barrier();  // all loads landed, all tiles consumed: stage memory is free
    f32x4* xch = reinterpret_cast<f32x4*>(smem) + lane;
    f32x2* ml = reinterpret_cast<f32x2*>(reinterpret_cast<float*>(smem) + ML) + qw * KW * 64 + lane;
    ml[kw * 64] = f32x2{m_run, l_all};
    // slot (query-wave, owner, source): a wave leaves the shares of the others
#pragma unroll
    for (int o = 0; o < KW; ++o) {
      f32x4 share[OWN / 4];
#pragma unroll
      for (int i = 0; i < OWN; ++i) share[i >> 2][i & 3] = acc_o[(o * OWN + i) >> 4][(o * OWN + i) & 15];
      if (o == kw) {
#pragma unroll
        for (int i = 0; i < OWN / 4; ++i) own[i] = share[i];
      } else {
        f32x4* slot = xch + ((qw * KW + o) * (KW - 1) + (kw < o ? kw : kw - 1)) * (OWN / 4) * 64;
#pragma unroll
        for (int i = 0; i < OWN / 4; ++i) slot[i * 64] = share[i];
      }
    }
    __syncthreads();
    f32x2 stat[KW];
#pragma unroll
    for (int o = 0; o < KW; ++o) stat[o] = ml[o * 64];
    m_run = stat[0][0];
#pragma unroll
    for (int o = 1; o < KW; ++o) m_run = fmaxf(m_run, stat[o][0]);
    l_all = 0.f;
    f32x4 sum[OWN / 4];
#pragma unroll
    for (int i = 0; i < OWN / 4; ++i) sum[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int o = 0; o < KW; ++o) {
      const float scale = __builtin_amdgcn_exp2f(stat[o][0] - m_run);
      l_all += stat[o][1] * scale;
      const f32x4* slot = xch + ((qw * KW + kw) * (KW - 1) + (o < kw ? o : o - 1)) * (OWN / 4) * 64;
#pragma unroll
      for (int i = 0; i < OWN / 4; ++i) sum[i] += (o == kw ? own[i] : slot[i * 64]) * scale;
    }
#pragma unroll
    for (int i = 0; i < OWN / 4; ++i) own[i] = sum[i];
  } else {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
    for (int i = 0; i < OWN; ++i) own[i >> 2][i & 3] = acc_o[i >> 4][i & 15];
  }

  // ---- keys cut over workgroups: leave (max, sum, O) at device scope (sc1); the last workgroup to
  // arrive at the block merges all parts in their order.  Nobody waits for anybody. ----
  if (n_parts > 1) {
    constexpr int kDeviceScope = 16;                            // cache policy sc1
    constexpr int kRow = REGS + 2;                              // floats per lane
    constexpr int kSlot = QW * 64 * kRow * 4;                   // bytes of a part
    const auto parts = __builtin_amdgcn_make_buffer_rsrc(p.part_out + (long)block * n_parts * (kSlot / 4), 0, n_parts * kSlot, 0x00027000);
    const int own_off = qw * (64 * kRow * 4) + kw * (OWN / 4) * 1024 + lane * 16;
    const int ml_off = qw * (64 * kRow * 4) + REGS / 4 * 1024 + lane * 8;
    if (valid) {
#pragma unroll
      for (int i = 0; i < OWN / 4; ++i)
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, own[i]), parts, part * kSlot + own_off + i * 1024, 0, kDeviceScope);
      const f32x2 ml = {m_run, l_all};
      if (kw == 0) __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, ml), parts, part * kSlot + ml_off, 0, kDeviceScope);
    }
    wait_all_and_barrier();
    int* last = reinterpret_cast<int*>(smem);
    if (tid == 0) *last = arrive_last(p.part_count + block, n_parts);
    __syncthreads();
    if (!*last) return;
    if (valid) {
      m_run = -INFINITY;
      l_all = 0.f;
#pragma unroll
      for (int i = 0; i < OWN / 4; ++i) own[i] = f32x4{0.f, 0.f, 0.f, 0.f};
      for (int q = 0; q < n_parts; ++q) {
        const f32x2 ml = __builtin_bit_cast(f32x2, __builtin_amdgcn_raw_buffer_load_b64(parts, q * kSlot + ml_off, 0, kDeviceScope));
        f32x4 v[OWN / 4];
#pragma unroll
        for (int i = 0; i < OWN / 4; ++i)
          v[i] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(parts, q * kSlot + own_off + i * 1024, 0, kDeviceScope));
        const float m_new = fmaxf(m_run, ml[0]);
        const float sa = __builtin_amdgcn_exp2f(m_run - m_new), sb = __builtin_amdgcn_exp2f(ml[0] - m_new);
        m_run = m_new;
        l_all = l_all * sa + ml[1] * sb;
#pragma unroll
        for (int i = 0; i < OWN / 4; ++i) own[i] = own[i] * sa + v[i] * sb;
      }
    }
  }
  if (!valid) return;
  const float inv = 1.0f / l_all;
  asm volatile("" : "+v"(tok));  // (one register until here, or the compiler forms the address in front of the loop)
  // registers 4 i .. 4 i + 3 of a lane are channels 8 i + 4 half ..
  bf16_t* orow = p.out + (long)tok * p.d + h * DH + kw * (OWN / 4) * 8 + half * 4;
#pragma unroll
  for (int i = 0; i < OWN / 4; ++i) {
    bf16x4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = (bf16_t)(own[i][e] * inv);
    *reinterpret_cast<bf16x4*>(orow + i * 8) = o;
  }
}

// Maximum over the lanes L, L ^ 16, L ^ 32 and L ^ 48.  (The swap's words are copied before they are taken for floats:
// __builtin_bit_cast of an element of a vector reads the first one.)
__device__ __forceinline__ float quarters_max(float x) {
  const unsigned own = __builtin_bit_cast(unsigned, x);
  const auto rows = __builtin_amdgcn_permlane16_swap(own, own, false, false);
  const unsigned even = rows[0], odd = rows[1];
  const unsigned pair = __builtin_bit_cast(unsigned, fmaxf(__builtin_bit_cast(float, even), __builtin_bit_cast(float, odd)));
  const auto halves = __builtin_amdgcn_permlane32_swap(pair, pair, false, false);
  const unsigned low = halves[0], high = halves[1];
  return fmaxf(__builtin_bit_cast(float, low), __builtin_bit_cast(float, high));
}

// XOR applied to the 16-byte chunk index of a K row / V row of attn_wide.  K fragment: 16 rows at one chunk; V
// fragment by transpose read: 8 rows at 32 bytes are read at a time.  Linear over the bits of the key.
__device__ __forceinline__ constexpr int wide_k_swizzle(int key) { return key & 15; }
__device__ __forceinline__ constexpr int wide_v_swizzle(int key) { return (key & 3) << 2 | (key >> 2 & 1) << 1; }
template <int KW>
constexpr int wide_smem_bytes() {  // two stages of K and of V, a tile of 64 keys of 128 channels per key-wave in each
  return 2 * KW * 2 * 64 * 128 * 2;
}

// A block of 32 QW query rows of heads of 128 channels, QW x KW waves: wave (qw, kw) owns 32 rows and every KW-th tile
// of 64 keys.  Arguments as for attn_block.
// What bounds it is the issue of a SIMD and power.  In step, the two waves of a SIMD multiplied, then both took their
// exponentials, and the matrix cores were idle for half of the time (0.52 M of 1.2 M cycles at 8 x 2048 tokens of 32 heads).
//   * Subtiles of 32 keys: while the logits of one are multiplied, the softmax of the one before and the value product
//     of the one before that run, an MFMA or two, an exponential, fragment reads, and so on, in one instruction stream.  Fragments
//     are read three MFMA groups ahead; the barrier of a step lies behind its last fragment, the first ones of the next
//     step follow it, so a step ends without an empty pipe.
//   * No maximum of every tile: the reference exponent of a row moves when a lane's sum of probabilities says so.
//   * v_mfma_f32_16x16x32_bf16, as in the large projections: the same loop with 32 x 32 x 16 has 10 % fewer cycles, at 1.8 GHz for 1.9
//     (of 2.4), and takes up to 10 % longer (and 30 registers more).
//   * QW = 4, KW = 1: two workgroups of four waves per CU, out of step with each other, one multiplies while the other
//     waits at its barrier or starts and ends.  One workgroup of eight waves (256 rows) pulls half as much from the L2 and is
//     slower all the same wherever sequences are short (when it was chosen: 3 x 777 tokens 56.9 us, two workgroups 46.5; 16 x
//     256 34.4 and 31.6; 8 x 2048 510 and 511; 1 x 4096 233 and 240).
// us, before (32 x 32 x 16, logits, softmax and values one after the other, 256 rows) and now, 32 heads, random inputs, one card: 8 x
// 2048 561 and 534 (1.03 PFLOP/s; in a step, by card, 540 to 570), 1 x 4096 260 and 247, 3 x 777 58.4 and 47.5, 16 x 256 36.0 and
// 32.1; KW = 2, 1 x 1024 23.3 and 22.2.  Heads of 64 channels
// keep attn_block, whose 120 registers let four waves share a SIMD: they have half of the MFMAs per exponential (8 x 2048 of
// 32 such heads 283 us, with this loop 282 to 325; 1 x 4096 142 and 150).
// Not faster: loads between the MFMAs instead of in a row behind the barrier (2 to 6 % slower), four stages (5 % slower),
// s_setprio around the MFMAs.
template <int QW, int KW>
__device__ __forceinline__ void attn_wide(const AttnDev& p, int b, int h, int qt, int cnt, int off,
                                          unsigned char* smem, const int tid) {
  constexpr int DH = 128, TK = 64, NW = QW * KW;
  constexpr int ROWB = DH * 2;                     // bytes per K or V row of one head (and a divisor of a token's, as the chunk XOR needs)
  constexpr int CPR = DH / 8;                      // 16-byte chunks per row
  constexpr int RPL = 64 / CPR;                    // rows covered by one wave load
  constexpr int TILE_BYTES = TK * ROWB;
  constexpr int KSTAGE = KW * TILE_BYTES;          // K (or V) of a stage
  constexpr int KL = KSTAGE / 1024 / NW;           // wave loads of K (or V) per step
  constexpr int CB = DH / 16;                      // 16-channel blocks of the output
  constexpr int NP = CB;                           // fragments of K, and of V, that a subtile takes
  constexpr int AHEAD = 3, RING = AHEAD + 1;       // fragments read ahead of their MFMAs
  // The reference exponent of a row moves to a maximum that is 2^grow above it, looked for where a lane's sum of probabilities
  // exceeds limit.  8 as in attn_block: a probability is at most 256, and times a value of up to 1e36 finite.
  const float grow = KW == 1 ? p.grow : 8.f, limit = KW == 1 ? p.limit : 256.f;
  static_assert(KSTAGE / 1024 % NW == 0 && NP % RING == 0, "loads and fragments must divide");
  using Yes = std::true_type;
  using No = std::false_type;
  using S0 = std::integral_constant<int, 0>;
  using S1 = std::integral_constant<int, 1>;

  const int T = p.seq;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // (a scalar: M0 addressing)
  const int qw = (unsigned)wave % QW, kw = (unsigned)wave / QW;
  const int l16 = lane & 15, kq = lane >> 4;

  // the query rows of this lane: 16 r + l16 of the wave's
  const bool any_row = qt * (32 * QW) + qw * 32 < cnt;  // (the same in all lanes: a wave without rows only loads)
  int tok[2];
  bool valid[2];
  bf16x8 qf[2][DH / 32];
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    const int j = qt * (32 * QW) + qw * 32 + r * 16 + l16;
    valid[r] = j < cnt;
    const int jc = valid[r] ? j : cnt - 1;
    tok[r] = p.idx ? p.idx[off + jc] : off + jc;
  }
#pragma unroll
  for (int r = 0; r < 2; ++r)
#pragma unroll
    for (int ks = 0; ks < DH / 32; ++ks)
      qf[r][ks] = *reinterpret_cast<const bf16x8*>(p.q + (long)tok[r] * p.d + h * DH + ks * 32 + kq * 8);

  const int n_tiles = (T + TK - 1) / TK, n_steps = (n_tiles + KW - 1) / KW;

  // ---- global -> LDS: two stages of K, two of V; a stage holds the tiles of the key-waves, a row of 1 KiB loads per wave ----
  const bf16_t* kbase = p.k + (long)b * T * p.d + h * DH;
  const bf16_t* vbase = p.v + (long)b * T * p.d + h * DH;
  const unsigned row_bytes = (unsigned)p.d * 2;
  const unsigned key0 = (unsigned)wave * KL * RPL + (unsigned)lane / CPR;  // key of this lane's first load at step 0
  // (the chunk XOR of a key is that of the lane's first key and that of the distance)
  const unsigned k_chunk = ((unsigned)lane % CPR ^ wide_k_swizzle(key0)) * 16, v_chunk = ((unsigned)lane % CPR ^ wide_v_swizzle(key0)) * 16;
  const unsigned k_src = key0 * row_bytes + k_chunk, v_src = key0 * row_bytes + v_chunk;
  const unsigned lds0 = (unsigned)(size_t)(lptr_t)smem;
  auto load_tiles = [&](auto is_v, int step) __attribute__((always_inline)) {
    constexpr bool V = decltype(is_v)::value;
    const int k0 = step * (KW * TK);
    const bf16_t* from = (V ? vbase : kbase) + (long)k0 * p.d;
    const unsigned to = lds0 + (V ? 2 * KSTAGE : 0) + (step & 1) * KSTAGE + wave * KL * 1024;
    auto load = [&](unsigned at, int i) __attribute__((always_inline)) {
      asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(at), "s"(from), "{m0}"(to + i * 1024) : "memory");
    };
#define DARE_SWZ(i) ((V ? wide_v_swizzle((i) * RPL) : wide_k_swizzle((i) * RPL)) * 16)
    if (k0 + KW * TK > T) {  // keys past the end re-read the last one
#pragma unroll
      for (int i = 0; i < KL; ++i) {
        const unsigned key = key0 + i * RPL, end = T - 1 - k0;
        load((key < end ? key : end) * row_bytes + ((V ? v_chunk : k_chunk) ^ DARE_SWZ(i)), i);
      }
    } else {
#pragma unroll
      for (int i = 0; i < KL; ++i) load(((V ? v_src : k_src) ^ DARE_SWZ(i)) + i * RPL * row_bytes, i);
    }
#undef DARE_SWZ
  };
  // Publishes K of step + 1 and V of step; every wave has read K of step and V of step - 1, whose stages are filled again
  auto next_tiles = [&](int step) __attribute__((always_inline)) {
    wait_vmcnt_and_barrier<0>();
    if (step + 2 < n_steps) load_tiles(No{}, step + 2);
    if (step + 1 < n_steps) load_tiles(Yes{}, step + 1);
  };

  // ---- fragments ----
  // K fragment j: keys 16 (j & 1) + l16, channels 32 (j / 2) + 8 kq ..
  // V fragment j, by transpose read: channel 16 j + l16, keys 4 kq .. +3 and 16 + 4 kq .. +3.  Lane i of a group of 16 gives
  // the address of key i / 4 of the run, channels 4 (i % 4) .. of the block.
  typedef const __attribute__((address_space(3))) bf16x8* lds_frag_t;
  unsigned k_at[NP / 2], v_at;
#pragma unroll
  for (int ks = 0; ks < NP / 2; ++ks)
    k_at[ks] = lds0 + kw * TILE_BYTES + l16 * ROWB + ((ks * 4 + kq) ^ wide_k_swizzle(l16)) * 16;
  {
    const int key = kq * 4 + (l16 >> 2);
    v_at = lds0 + 2 * KSTAGE + kw * TILE_BYTES + key * ROWB + ((l16 >> 1 & 1) ^ wide_v_swizzle(key)) * 16 + (l16 & 1) * 8;
  }
  bf16x8 kf[RING], vf[RING];
  auto read_k = [&](int j, int sub) __attribute__((always_inline)) {
    // (keys 16 apart have one chunk XOR)
    kf[j % RING] = *(lds_frag_t)(k_at[j / 2] + (sub * 32 + (j & 1) * 16) * ROWB);
  };
  auto read_v = [&](int j, int sub) __attribute__((always_inline)) {
    const unsigned at = lds0 + ((v_at - lds0) ^ j * 32) + sub * 32 * ROWB;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(at));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(at + 16 * ROWB));
    vf[j % RING] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };

  f32x4 acc[CB][2];         // [channel block][row block]: channels 4 kq .. of the block
  f32x4 sc[2][2][2];        // logits of two subtiles, [set][row block][16 keys]: keys 4 kq ..
  bf16x8 pf[2][2];          // probabilities of two subtiles, [set][row block]
  float m_run[2] = {-INFINITY, -INFINITY}, l_run[2] = {0.f, 0.f};
#pragma unroll
  for (int c = 0; c < CB; ++c)
#pragma unroll
    for (int r = 0; r < 2; ++r) acc[c][r] = f32x4{0.f, 0.f, 0.f, 0.f};

  // ---- softmax of a subtile: logit n = 8 row block + key slot ----
  const bf16x2 ones = {(bf16_t)1.0f, (bf16_t)1.0f};
  float e0 = 0.f, e1 = 0.f;
  auto exp_one = [&](const f32x4 (&x)[2][2], int n) __attribute__((always_inline)) {
    const float v = __builtin_amdgcn_exp2f(fmaf(x[n >> 3][n >> 2 & 1][n & 3], p.scale_log2, -m_run[n >> 3]));
    if (n & 1) e1 = v; else e0 = v;
  };
  // rounded for the value product; the row sum is taken over the probabilities as rounded (v_dot2: += both), so
  // numerator and denominator carry the same rounding
  auto round_pair = [&](bf16x8 (&pr)[2], int n, float (&sum)[2]) __attribute__((always_inline)) {
    const f32x2 v = {e0, e1};
    const bf16x2 pb = __builtin_convertvector(v, bf16x2);
    sum[n >> 3] = __builtin_amdgcn_fdot2_f32_bf16(pb, ones, sum[n >> 3], false);
    pr[n >> 3][n & 7] = pb[0];
    pr[n >> 3][(n & 7) + 1] = pb[1];
  };
  auto mask_keys = [&](f32x4 (&x)[2][2], int kv0) __attribute__((always_inline)) {  // keys past the end
#pragma unroll
    for (int n = 0; n < 8; ++n)
      if (kv0 + (n >> 2) * 16 + kq * 4 + (n & 3) >= T) x[0][n >> 2][n & 3] = x[1][n >> 2][n & 3] = -INFINITY;
  };
  // The reference exponents of a block of 16 rows move to the maxima of this subtile, which is scored again, and of the other
  // set's, the next subtile (keys past the end are copies of the last one there), where those are far enough above.  Any reference
  // gives the same result up to rounding (O and the row sum share it), so they only move when probabilities grow large, which a
  // lane's sum of them tells without the maximum of every subtile.  FIRST: there is none yet.
  //   * Steep logits: nearly every subtile has a row that grows, and a move takes a wave 350 cycles per block.  Hence one block
  //     alone, and the next subtile as well, which then seldom moves them again (us by standard deviation of the logits in nats, 1.6, 9,
  //     25; attn_block, both blocks and this subtile, now: 1 x 1024 tokens of 32 heads 23.6 24.8 24.9, 22.3 29.2 30.3, 22.4 26.7 26.6; 8
  //     x 2048 581 612 608, 540 604 620, 539 599 606; 3 x 777 58.2 61.0 61.2, 47.2 54.5 55.0, 47.1 55.2 56.1).  A row with less growth than
  //     grow stays where it is: moving it along is 2 to 5 % faster, but leaves long rows with fewer exact largest probabilities
  //     (1 x 4096 tokens, logits of 4 nats, error 1.883e-3 for 1.864e-3).
  //   * The largest probability of a tile that the reference is taken from is 1, without a rounding, and rows are the nearer to their
  //     exact value the more of their tiles have that.  So the first reference is the maximum of the wave's first tile, and one wave
  //     in the place of two (attn_second_reference) moves to that of its second tile too, also down (by 8 at most), and moves with less
  //     growth, to any maximum above.  Error against float64 in 10^-3 with the first subtile's maximum, the first tile's, this,
  //     and with two key-waves: 129 keys 2.18, 2.12, 1.99, 1.99; 300 keys 2.25, 2.23, 2.16, 2.16; with logits of 4 nats, first tile and
  //     second, this, two key-waves: 512 keys 1.80, 1.77, 1.83; 2560 keys 1.87, 1.83, 1.85; 3840 keys 1.88, 1.84, 1.85.
  auto move_reference = [&](auto r_c, const f32x4 (&x)[2][2], const f32x4 (&next)[2][2], bf16x8 (&pr)[2], float (&sum)[2], auto first_c, bool second) __attribute__((always_inline)) {
    constexpr int r = decltype(r_c)::value;
    float top = x[r][0][0];
#pragma unroll
    for (int n = 1; n < 8; ++n) top = fmaxf(top, x[r][n >> 2][n & 3]);
#pragma unroll
    for (int n = 0; n < 8; ++n) top = fmaxf(top, next[r][n >> 2][n & 3]);
    top = quarters_max(top) * p.scale_log2;  // scale > 0
    const float moved = second ? fmaxf(top, m_run[r] - 8.f) : top > m_run[r] + grow ? top : m_run[r];
    const float m_new = fmaxf(moved, -__FLT_MAX__);  // (finite: logits of -infinity have probability 0)
    if constexpr (!decltype(first_c)::value) {
      const float alpha = __builtin_amdgcn_exp2f(m_run[r] - m_new);
      l_run[r] *= alpha;
#pragma unroll
      for (int c = 0; c < CB; ++c) acc[c][r] *= alpha;
    }
    m_run[r] = m_new;
    sum[r] = 0.f;
#pragma unroll
    for (int n = 8 * r; n < 8 * r + 8; n += 2) {
      exp_one(x, n);
      exp_one(x, n + 1);
      round_pair(pr, n, sum);
    }
  };

  // One subtile period.  QK: logits of subtile u (into sc[S ^ 1]); SM: softmax of u - 1 (sc[S], into pf[S]); PV: values of
  // u - 2 (pf[S ^ 1]); three that do not depend on each other, one after the other in small pieces, so that MFMAs,
  // exponentials and LDS reads run side by side.  MORE: a period follows.
  auto period = [&](auto s_c, auto qk_c, auto sm_c, auto pv_c, auto more_c, int step) __attribute__((always_inline)) {
    constexpr int S = decltype(s_c)::value, SUB = S ^ 1;  // SUB: subtile of its tile, of K and V alike
    constexpr bool QK = decltype(qk_c)::value, SM = decltype(sm_c)::value, PV = decltype(pv_c)::value;
    constexpr bool MORE = decltype(more_c)::value, EDGE = SUB == 1;  // EDGE: the step's tiles end here
    constexpr int LPP = 16 / NP;        // logits per fragment
    constexpr int SPLIT = NP - AHEAD;   // fragment behind whose MFMAs the step's last ones are in registers
    float sum[2] = {0.f, 0.f};
    auto softmax = [&](int first, int last) __attribute__((always_inline)) {
      if constexpr (SM) {
#pragma unroll
        for (int n = first; n < last; ++n) {
          if (n % 2 == 0 && n > 0) round_pair(pf[S], n - 2, sum);
          exp_one(sc[S], n);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    };
#pragma unroll
    for (int j = 0; j < NP; ++j) {
      __builtin_amdgcn_sched_barrier(0);
      const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
      f32x4 (&x)[2][2] = sc[S ^ 1];
      if constexpr (QK) x[0][j & 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[j % RING], qf[0][j / 2], j < 2 ? zero : x[0][j & 1], 0, 0, 0);
      softmax(j * LPP, j * LPP + LPP / 2);
      if constexpr (QK) x[1][j & 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[j % RING], qf[1][j / 2], j < 2 ? zero : x[1][j & 1], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (PV) acc[j][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[j % RING], pf[S ^ 1][0], acc[j][0], 0, 0, 0);
      softmax(j * LPP + LPP / 2, (j + 1) * LPP);
      if constexpr (PV) acc[j][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[j % RING], pf[S ^ 1][1], acc[j][1], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      if (j + AHEAD < NP) {
        if constexpr (QK) read_k(j + AHEAD, SUB);
        if constexpr (PV) read_v(j + AHEAD, SUB);
      } else if constexpr (MORE && !EDGE) {
        if constexpr (QK) read_k(j + AHEAD - NP, 1);
        if constexpr (PV) read_v(j + AHEAD - NP, 1);
      }
      if constexpr (EDGE && MORE) {
        if (j == SPLIT) {  // all of the step's fragments are in registers: its stages may be filled again
          if constexpr (SM) asm volatile("" : "+v"(sum[0]), "+v"(sum[1]), "+v"(e0), "+v"(e1));  // (what is done so far stays in front of the branches)
          next_tiles(step);
#pragma unroll
          for (int i = 0; i < NP / 2; ++i) k_at[i] = lds0 + ((k_at[i] - lds0) ^ KSTAGE);
          if constexpr (PV) v_at = lds0 + ((v_at - lds0) ^ KSTAGE);
        }
        if (j > SPLIT) {
          const int from = AHEAD * (j - SPLIT - 1) / (AHEAD - 1), to = AHEAD * (j - SPLIT) / (AHEAD - 1);
#pragma unroll
          for (int i = from; i < to; ++i) {
            read_k(i, 0);
            read_v(i, 0);
          }
        }
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (SM) {
      round_pair(pf[S], 14, sum);
      const bool second = KW == 1 && EDGE && step == p.second;
      const float above = second ? -1.f : limit;  // (-1: whatever the sums are)
      if (__any(fmaxf(sum[0], sum[1]) > above)) {
        if (__any(sum[0] > above)) move_reference(S0{}, sc[S], sc[S ^ 1], pf[S], sum, No{}, second);
        if (__any(sum[1] > above)) move_reference(S1{}, sc[S], sc[S ^ 1], pf[S], sum, No{}, second);
      }
      l_run[0] += sum[0];
      l_run[1] += sum[1];
    }
  };

  // the wave's tiles; all waves load, and join the barrier of every step
  int mine = (n_tiles - kw + KW - 1) / KW;
  mine = !any_row || mine < 0 ? 0 : (mine < n_steps ? mine : n_steps);
  auto key_of = [&](int step) __attribute__((always_inline)) { return (step * KW + kw) * TK; };
  load_tiles(No{}, 0);
#pragma unroll
  for (int r = 0; r < 2; ++r)
#pragma unroll
    for (int ks = 0; ks < DH / 32; ++ks) asm volatile("" : "+v"(qf[r][ks]));  // (waits for the queries and these keys)
  wait_vmcnt_and_barrier<0>();
  load_tiles(Yes{}, 0);
  if (n_steps > 1) load_tiles(No{}, 1);
  if (mine > 0) {
#pragma unroll
    for (int j = 0; j < AHEAD; ++j) read_k(j, 0);
    period(S1{}, Yes{}, No{}, No{}, Yes{}, 0);
    period(S0{}, Yes{}, No{}, No{}, Yes{}, 0);
    if (key_of(0) + 64 > T) {
      mask_keys(sc[0], key_of(0));
      mask_keys(sc[1], key_of(0) + 32);
    }
    move_reference(S0{}, sc[0], sc[1], pf[0], l_run, Yes{}, false);
    move_reference(S1{}, sc[0], sc[1], pf[0], l_run, Yes{}, false);
    for (int step = 1; step < mine; ++step) {
      period(S1{}, Yes{}, Yes{}, Yes{}, Yes{}, step);
      if (key_of(step) + 32 > T) mask_keys(sc[0], key_of(step));
      period(S0{}, Yes{}, Yes{}, Yes{}, Yes{}, step);
    }
    if (mine > 1 && key_of(mine - 1) + 64 > T) mask_keys(sc[1], key_of(mine - 1) + 32);
    period(S1{}, No{}, Yes{}, Yes{}, Yes{}, mine);
    period(S0{}, No{}, No{}, Yes{}, No{}, mine);
  }
  for (int step = mine; step < n_steps; ++step) next_tiles(step);

#pragma unroll
  for (int r = 0; r < 2; ++r) {
    l_run[r] += __shfl_xor(l_run[r], 16, 64);
    l_run[r] += __shfl_xor(l_run[r], 32, 64);
  }

  // ---- merge the key-waves: every one merges, and stores, its share of the channel blocks ----
  constexpr int OWN = CB / KW;  // channel blocks of a wave
  f32x4 own[OWN][2];            // blocks kw OWN ..
  if constexpr (KW > 1) {
    constexpr int ML = QW * KW * (KW - 1) * OWN * 2 * 64 * 16;  // bytes of the shares; behind them (max, sum) of every wave
    static_assert(ML + QW * KW * 64 * 16 <= wide_smem_bytes<KW>(), "the merge area must fit into the stage memory");
    wait_all_and_barrier();  // all loads landed, all tiles consumed: stage memory is free
    f32x4* xch = reinterpret_cast<f32x4*>(smem) + lane;
    f32x4* ml = reinterpret_cast<f32x4*>(smem + ML) + qw * KW * 64 + lane;
    ml[kw * 64] = f32x4{m_run[0], l_run[0], m_run[1], l_run[1]};
    // slot (query-wave, owner, source): a wave leaves the shares of the others
#pragma unroll
    for (int o = 0; o < KW; ++o)
      if (o == kw) {
#pragma unroll
        for (int i = 0; i < OWN; ++i)
#pragma unroll
          for (int r = 0; r < 2; ++r) own[i][r] = acc[o * OWN + i][r];
      } else {
        f32x4* slot = xch + ((qw * KW + o) * (KW - 1) + (kw < o ? kw : kw - 1)) * OWN * 2 * 64;
#pragma unroll
        for (int i = 0; i < OWN; ++i)
#pragma unroll
          for (int r = 0; r < 2; ++r) slot[(i * 2 + r) * 64] = acc[o * OWN + i][r];
      }
    __syncthreads();
    f32x4 stat[KW];
#pragma unroll
    for (int o = 0; o < KW; ++o) stat[o] = ml[o * 64];
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      float m = stat[0][2 * r], l = 0.f;
#pragma unroll
      for (int o = 1; o < KW; ++o) m = fmaxf(m, stat[o][2 * r]);
      f32x4 sum[OWN];
#pragma unroll
      for (int i = 0; i < OWN; ++i) sum[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int o = 0; o < KW; ++o) {
        const float scale = __builtin_amdgcn_exp2f(stat[o][2 * r] - m);
        l += stat[o][2 * r + 1] * scale;
        const f32x4* slot = xch + ((qw * KW + kw) * (KW - 1) + (o < kw ? o : o - 1)) * OWN * 2 * 64;
#pragma unroll
        for (int i = 0; i < OWN; ++i) sum[i] += (o == kw ? own[i][r] : slot[(i * 2 + r) * 64]) * scale;
      }
#pragma unroll
      for (int i = 0; i < OWN; ++i) own[i][r] = sum[i];
      l_run[r] = l;
    }
  } else {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
    for (int i = 0; i < OWN; ++i)
#pragma unroll
      for (int r = 0; r < 2; ++r) own[i][r] = acc[i][r];
  }
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    if (!valid[r]) continue;
    const float inv = 1.0f / l_run[r];
    asm volatile("" : "+v"(tok[r]));  // (one register until here, or the compiler forms the address in front of the loop)
    bf16_t* row = p.out + (long)tok[r] * p.d + h * DH + kw * OWN * 16 + kq * 4;
#pragma unroll
    for (int i = 0; i < OWN; ++i) {
      bf16x4 o;
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = (bf16_t)(own[i][r][e] * inv);
      *reinterpret_cast<bf16x4*>(row + i * 16) = o;
    }
  }
}

// A workgroup without a query block of its own, one of `helpers` of its (sequence, head) on the same
// XCD: reads the keys and values behind the first step once, in the order of the steps, so that the
// blocks, whose two stages in flight would wait for every line at the latency of HBM (60 GB/s per CU), find
// them in the XCD's L2 (158 GB/s).  (Steps over 1 x 1024 tokens of 32 heads whose caches come from HBM: 4
// refreshed rows 65.0 -> 60.6 us, 205 rows 89.4 -> 87.9.  The weights of the output projection read ahead
// here as well: 62.9 and 86.9, not kept.)
template <int DH, int NW>
__device__ __forceinline__ void read_ahead(const AttnDev& p, int b, int h, int helper, int helpers, unsigned char* smem) {
  constexpr int CPR = DH / 8, RPL = 64 / CPR;  // 16-byte chunks per row, rows covered by one wave load
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const long at = (long)b * p.seq * p.d + h * DH + (lane % CPR) * 8;
  for (int u = 128 / RPL * 2 + helper * NW + wave; u < (p.seq + RPL - 1) / RPL * 2; u += helpers * NW) {
    int key = (u >> 1) * RPL + lane / CPR;
    key = key < p.seq ? key : p.seq - 1;
    load_to_lds((u & 1 ? p.v : p.k) + at + (long)key * p.d, smem + wave * 1024);  // (nobody reads it)
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

template <int DH, int QW, int KW, int TK, int NST>
__global__ void __launch_bounds__(QW* KW * 64, 2) attn_bf16_kernel(AttnDev p) {
  __shared__ __attribute__((aligned(1024))) unsigned char smem[attn_smem_bytes<DH, KW, TK, NST>()];
  // Workgroup ids are dealt round-robin to the 8 XCDs.  All query blocks of one
  // (sequence, head) are placed on the same XCD, so its K and V are fetched from HBM
  // once and re-read from that XCD's L2 by the other blocks.
  AttnPlace at = {blockIdx.x >> 3, 0};
  if (p.n_qt > 1) at = attn_place(at.pair, (unsigned)(p.n_pairs + 7) >> 3, p.n_qt, p.turn);
  const int pair = at.pair * 8 + (blockIdx.x & 7), qt = at.block;
  if (pair >= p.n_pairs) return;
  const int b = pair / p.n_heads, h = pair % p.n_heads;
  int cnt, off;
  if (p.idx) {
    off = p.sel_off[b];
    cnt = p.sel_off[b + 1] - off;
  } else {
    off = b * p.seq;
    cnt = p.seq;
  }
  if (qt * (32 * QW) >= cnt) {
    const int blocks = (cnt + 32 * QW - 1) / (32 * QW);
    if (blocks > 0 && qt < p.at_once)
      read_ahead<DH, QW * KW>(p, b, h, qt - blocks, (p.at_once < p.n_qt ? p.at_once : p.n_qt) - blocks, smem);
    return;
  }
  if constexpr (TK == 64 && DH == 128) {
    static_assert(sizeof(smem) == wide_smem_bytes<KW>(), "the stage memory of attn_wide");
    attn_wide<QW, KW>(p, b, h, qt, cnt, off, smem, threadIdx.x);
  } else
    attn_block<DH, QW, KW, TK, NST>(p, b, h, qt, cnt, off, smem, threadIdx.x);
}

// Refreshed rows: how many of a sequence's tokens there are is known on the device only, so the
// grid is as many workgroups as run at once (kRowsGrid) and the query blocks are laid out from the
// counts: 64 rows per block while that gives at most one block per workgroup, else 128 (a K/V tile then
// feeds twice the rows: 3 x 777 tokens, 194 rows each: 24 against 35 us; 1 x 1024, 205 rows: 18 us against
// 21 us the other way round), whose last round runs as blocks of 64 rows where it would leave half of the workgroups
// idle (attn_whole_blocks; heads of 128 channels).  Few blocks over long sequences leave most CUs without one and the others
// with a long chain of key steps: their keys are cut over workgroups, in parts of at least kPartSteps
// steps (the hand-over costs about as much as four).
// Blocks are numbered by sequence, head, part, query block; consecutive ones, which share keys,
// go to one XCD (workgroup ids are dealt round-robin to the 8 XCDs).
// A wave holds the blocks of 64 sequences, a sequence per lane, summed up along the lanes: the
// sequence of a block is a ballot away, and a workgroup, whose blocks come in ascending order, walks
// the sequences twice in all (lane by lane it was 75 ns per sequence and block).
// v / n for 0 <= v < 2^24, n > 0, the same in all lanes (a handful of instructions where the exact
// division takes 40)
__device__ __forceinline__ int small_div(int v, int n) {
  int q = __builtin_amdgcn_readfirstlane((int)((float)v * __builtin_amdgcn_rcpf((float)n)));
  const int r = v - q * n;
  if (r >= n) ++q;
  if (r < 0) --q;
  return q;
}
// sum over the lanes up to and including this one
__device__ __forceinline__ int wave_prefix_sum(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);  // row_shr 1, 2, 4, 8: within 16 lanes
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);  // row_bcast 15: lane 15 to row 1, 47 to row 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);  // row_bcast 31: lane 31 to rows 2 and 3
  return v;
}
// Workgroups that run at once: one per CU (128 KB of LDS), two with 64 channels per head (64 KB)
template <int DH>
constexpr int kRowsGrid = DH == 64 ? 512 : 256;
template <int DH>
__global__ void __launch_bounds__(512, kRowsGrid<DH> / 128) attn_rows_bf16_kernel(AttnDev p) {
  __shared__ __attribute__((aligned(1024))) unsigned char smem[attn_smem_bytes<DH, 4, 32, 2>()];
  static_assert(attn_smem_bytes<DH, 4, 32, 2>() == attn_smem_bytes<DH, 2, 64, 2>(), "one stage memory for both blocks");
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  __builtin_assume(p.idx != nullptr);
  int off_l = 0, cnt_l = 0;  // the 64 sequences held: first list position and refreshed rows of c0 + lane
  auto hold = [&](int c0) __attribute__((always_inline)) {
    const int b = c0 + (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0));
    off_l = b < p.batch ? p.sel_off[b] : 0;
    cnt_l = b < p.batch ? p.sel_off[b + 1] - off_l : 0;
  };
  int narrow = 0, wide = 0;  // blocks of 64 and of 128 rows
  for (int c0 = 0; c0 < p.batch; c0 += 64) {
    hold(c0);
    narrow += __builtin_amdgcn_readlane(wave_prefix_sum((cnt_l + 63) >> 6), 63);
    wide += __builtin_amdgcn_readlane(wave_prefix_sum((cnt_l + 127) >> 7), 63);
  }
  narrow *= p.n_heads;
  wide *= p.n_heads;
  const bool is_wide = narrow > kRowsGrid<DH>;
  const int shift = is_wide ? 7 : 6, rows = 1 << shift, blocks = is_wide ? wide : narrow;
  const int steps = (p.seq + 127) >> 7;  // of 128 keys, in either block
  int n_parts = 1;
  if (p.part_out && blocks > 0 && steps >= kCutSteps) {
    const int room = small_div(kAttnParts, blocks), most = steps / kPartSteps;
    n_parts = room < most ? room : most;
    if (n_parts < 1) n_parts = 1;
  }
  const int total = blocks * n_parts, per_xcd = (total + 7) >> 3;
  int per_block = p.n_heads * n_parts;        // units per query block of a sequence
  int c0 = 0, before = 0;                     // sequences held, query blocks in front of them
  if (p.batch > 64) hold(0);
  int upto = wave_prefix_sum((cnt_l + rows - 1) >> shift);
  // Blocks of 128 rows that are left for a last round of at most half of the workgroups: two of 64 rows each instead
  const int slots = gridDim.x >> 3, whole = DH == 128 ? attn_whole_blocks(per_xcd, slots, is_wide) : per_xcd, n_slots = 2 * per_xcd - whole;
  for (int slot = blockIdx.x >> 3; slot < n_slots; slot += gridDim.x >> 3) {
    const bool halved = DH == 128 && slot >= whole;
    const int u = (blockIdx.x & 7) * per_xcd + (halved ? whole + ((slot - whole) >> 1) : slot);
    if (u >= total) break;
    // (or their reciprocals stay in vector registers, which the block needs)
    asm volatile("" : "+s"(n_parts), "+s"(per_block));
    // the sequence: first one up to whose end there are more than u units
    const int w = small_div(u, per_block);
    for (int held = __builtin_amdgcn_readlane(upto, 63); before + held <= w; held = __builtin_amdgcn_readlane(upto, 63)) {
      before += held;
      c0 += 64;
      hold(c0);
      upto = wave_prefix_sum((cnt_l + rows - 1) >> shift);
    }
    const int l = __builtin_ctzll(__ballot(before + upto > w));
    const int b = c0 + l, off = __builtin_amdgcn_readlane(off_l, l), cnt = __builtin_amdgcn_readlane(cnt_l, l);
    const int n_qt = (cnt + rows - 1) >> shift;
    // units in front of the sequence
    const int first = (before + __builtin_amdgcn_readlane(upto, l) - n_qt) * per_block, v = u - first;
    const int part_and_head = small_div(v, n_qt), qt = v - part_and_head * n_qt;
    const int h = small_div(part_and_head, n_parts), part = part_and_head - h * n_parts;
    // block number without the parts: what precedes this sequence, then head and query block
    const int block = small_div(first, n_parts) + h * n_qt + qt;
    // (a thread number that the compiler cannot trace back, nor keep: it would hold it, and what both
    // blocks derive from it, in registers that the blocks need)
    unsigned every = ~0u;
    asm volatile("" : "+s"(every));
    const int tid = wave * 64 + (int)__builtin_amdgcn_mbcnt_hi(every, __builtin_amdgcn_mbcnt_lo(every, 0));
    if (is_wide && !halved) {  // (more than kAttnParts / 2 blocks: one part each)
      if constexpr (DH == 128) {
        static_assert(sizeof(smem) == wide_smem_bytes<2>(), "the stage memory of attn_wide");
        attn_wide<4, 2>(p, b, h, qt, cnt, off, smem, tid);
      } else
        attn_block<DH, 4, 2, 64, 2>(p, b, h, qt, cnt, off, smem, tid);
    } else {
      int q = qt;
      if (halved) {
        q = 2 * qt + ((slot - whole) & 1);
        if (q * 64 >= cnt) continue;  // (the second half of a last block; this round is the last one)
      }
      attn_block<DH, 2, 4, 32, 2>(p, b, h, q, cnt, off, smem, tid, part, n_parts, block);
    }
    if (slot + (int)(gridDim.x >> 3) >= n_slots) break;
    hold(c0);  // (again, rather than in registers that the block needs)
    upto = wave_prefix_sum((cnt_l + rows - 1) >> shift);
    __syncthreads();  // the stage memory is reused
  }
}

template <int DH, int QW, int KW, int TK, int NST>
hipError_t launch_variant(AttnDev p, const AttnArgs& a, hipStream_t s) {
  p.n_heads = a.n_heads;
  p.n_pairs = a.batch * a.n_heads;
  p.n_qt = (attn_most_rows(a.seq, a.idx != nullptr, a.many_rows, a.active) + 32 * QW - 1) / (32 * QW);
  p.second = attn_second_reference(p.n_pairs, attn_most_rows(a.seq, a.idx != nullptr, a.many_rows, a.active)) ? 1 : 0;
  p.limit = p.second ? 32.f : 256.f;
  p.grow = p.second ? 0.f : 8.f;
  p.turn = attn_turn(p.n_pairs, a.idx != nullptr, a.many_rows);
  p.at_once = a.idx && !a.many_rows ? attn_at_once(p.n_pairs, a.seq, DH) : 0;
  const long grid = (long)((p.n_pairs + 7) / 8) * p.n_qt * 8;
  if (grid > 0x7fffffffL) return hipErrorInvalidValue;
  hipLaunchKernelGGL((attn_bf16_kernel<DH, QW, KW, TK, NST>), dim3((unsigned)grid), dim3(QW * KW * 64), 0, s, p);
  return hipGetLastError();
}

template <int DH>
hipError_t launch_dh(const AttnDev& p, const AttnArgs& a, hipStream_t s) {
  switch (attn_route(a.batch, a.n_heads, a.seq, a.idx != nullptr, a.many_rows, a.parts.out != nullptr, DH, a.active)) {
    case AttnRoute::kNarrow: return launch_variant<DH, 2, 4, 32, 2>(p, a, s);
    case AttnRoute::kWide: return launch_variant<DH, 4, 2, 64, 2>(p, a, s);
    case AttnRoute::kTall: return launch_variant<DH, DH == 128 ? 4 : 8, 1, 64, 2>(p, a, s);
    case AttnRoute::kLaidOut: break;
  }
  AttnDev r = p;
  r.n_heads = a.n_heads;
  r.batch = a.batch;
  r.part_out = a.parts.out;
  r.part_count = a.parts.count;
  const long blocks = (long)a.batch * a.n_heads * ((a.seq + 63) / 64);  // with every row refreshed
  const bool cut = a.parts.out && attn_may_cut(a.seq);
  const long grid = cut || blocks >= kRowsGrid<DH> ? kRowsGrid<DH> : (blocks + 7) / 8 * 8;
  hipLaunchKernelGGL(attn_rows_bf16_kernel<DH>, dim3((unsigned)grid), dim3(512), 0, s, r);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_attn_bf16(const AttnArgs& a, hipStream_t s) {
  AttnDev p{};
  p.q = static_cast<const bf16_t*>(a.q);
  p.k = static_cast<const bf16_t*>(a.k);
  p.v = static_cast<const bf16_t*>(a.v);
  p.out = static_cast<bf16_t*>(a.out);
  p.idx = a.idx;
  p.sel_off = a.sel_off;
  p.seq = a.seq;
  p.d = a.n_heads * a.head_dim;
  p.scale_log2 = kLog2e / sqrtf((float)a.head_dim);
  if (a.head_dim == 128) return launch_dh<128>(p, a, s);
  if (a.head_dim == 64) return launch_dh<64>(p, a, s);
  return hipErrorInvalidValue;
}

}  // namespace dare
