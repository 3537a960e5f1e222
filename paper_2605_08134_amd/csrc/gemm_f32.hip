// fp32 path of the row-selected projection C[t, :] = A[t, :] . W (same contract as the
// bf16 kernel; Alg. 1 lines 2, 6-7, 11, Alg. 2 lines 2, 7, 11) on v_mfma_f32_16x16x4_f32.
//
// Fragments go from global memory straight into registers: lane L of a wave holds row L & 15
// and the four neighbouring k of chunk L >> 4, so one 16-byte load per 16 rows feeds four MFMAs
// (MFMA j multiplies element j of every chunk; A and W agree on that order).  The weight
// fragment is the first operand: a lane then owns one output row and four neighbouring columns.
//
// Every output is the sum of four sums over the quarters of k, added in order, whatever the
// tile shape: a row's projection does not depend on the number of rows or columns it is
// computed with, bit for bit (a query that did not change keeps a drift score of exactly 0
// across modes, which project it in launches of different width).
//
// What bounds it.  Small shapes (128 x 256 x 256): the latency of a workgroup, launch, one round
// of loads, sum, store.  Four waves take a quarter of k each, 4 x 16 k in flight per wave, and 16 x 16
// tiles give the most workgroups: 16.6 -> 3.8 us against a 64 x 64 LDS tile that walked k in steps of 16
// with two barriers each.  Larger shapes: the matrix pipe (157 TFLOP/s nominal; 117 reached)
// and the loads that feed it, hence 64 x 64 wave tiles, 64 MFMAs per 8 loads.  The four waves share the
// tile there too: four tiles of 64 x 64 per workgroup, every wave all of k, are no faster with many
// rows (1024 x 12288 x 4096 916 us against 880) and waste up to 127 rows of 128 with few.
#include "dare_common.h"

namespace dare {
namespace {

struct GemmF32Dev {
  const float* a;
  const float* wt;
  const int32_t* idx;
  const int32_t* m_dev;
  float* c0;
  float* c1;
  float* c2;
  float* c32;
  int lda, n, k, m_max, ldc, seg_n, c32_cols;
  const float* rope;
  int rope_cols, rope_dh, rope_seq;
  const uint8_t* sel_mask;  // row list made in the kernel, as in the bf16 path
  int sel_batch, sel_seq;
  int32_t* sel_idx_out;
  int32_t* sel_idx_out2;
  int32_t* sel_off_out;
  int32_t* sel_count_out;
};

// four neighbouring output columns col .. col + 3 (col a multiple of 4) of token tok
__device__ __forceinline__ void store4_f32(const GemmF32Dev& p, long tok, int col, f32x4 v) {
  const int seg = (col >= p.seg_n) + (col >= 2 * p.seg_n);
  float* cbase = seg == 0 ? p.c0 : (seg == 1 ? p.c1 : p.c2);
  if (p.c32 && col < p.c32_cols)  // the scored columns: before any rotation
    *reinterpret_cast<f32x4*>(p.c32 + tok * p.c32_cols + col) = v;
  if (!cbase) return;
  float v0 = v[0], v1 = v[1], v2 = v[2], v3 = v[3];
  if (p.rope && col < p.rope_cols) {
    const long at = (long)((unsigned)tok % (unsigned)p.rope_seq) * p.rope_dh + (unsigned)col % (unsigned)p.rope_dh;
    rope_rotate4(*reinterpret_cast<const f32x4*>(p.rope + at), v0, v1, v2, v3);
  }
  const f32x4 o = {v0, v1, v2, v3};
  *reinterpret_cast<f32x4*>(cbase + tok * p.ldc + (col - seg * p.seg_n)) = o;
}

// The refreshed-row list from the mask bytes, by every workgroup (256 threads) for itself; at most kSelMaxTokensF32
// tokens, four per thread, ascending.  The first workgroup also writes what a compaction kernel would.  Returns the count.
// (A launch less, for a few hundred bytes of work: steps of 1 x 128 tokens of hidden 256 21.9 -> 20.5 us, K/V reuse 21.9 ->
// 20.1; of 2 x 257 of 512 59.9 -> 56.5.  The score in the launch that projects its columns, as in bf16, is not: whole rows per
// workgroup leave 8 of 256 CUs to pull the weights, 7.1 us where projection and score take 3.8 and 3.1.)
__device__ __forceinline__ int derive_rows_f32(const GemmF32Dev& p, int32_t* list, int* wave_tot) {
  const int n_tok = p.sel_batch * p.sel_seq, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, t0 = tid * 4;
  bool z[4];
  int cnt = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint8_t reused = p.sel_mask[t0 + i < n_tok ? t0 + i : n_tok - 1];
    z[i] = t0 + i < n_tok && reused == 0;
    cnt += z[i];
  }
  int incl = cnt;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int up = __shfl_up(incl, o, 64);
    if (lane >= o) incl += up;
  }
  if (lane == 63) wave_tot[wave] = incl;
  __syncthreads();
  int rank = incl - cnt, total = 0;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    if (w < wave) rank += wave_tot[w];
    total += wave_tot[w];
  }
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if (z[i]) list[rank++] = t0 + i;
  __syncthreads();
  if (blockIdx.x == 0 && blockIdx.y == 0) {
    for (int r = tid; r < total; r += 256) {
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
    for (int b = tid; b <= p.sel_batch; b += 256) {
      const int off = before(b);
      p.sel_off_out[b] = off;
      if (p.sel_count_out && b < p.sel_batch) p.sel_count_out[b] = before(b + 1) - off;
    }
  }
  return total;
}

constexpr int kKParts = 4;  // quarters of k (k is a multiple of 64: whole steps of 16 each)

// Four waves on one tile of 16 TM x 16 TN, a quarter of k each, sums added through LDS.  UNR: steps of 16 k
// whose loads are in flight at once (registers allow one for 64 x 64, whose 64 MFMAs per step
// cover a load).
template <int TM, int TN, int UNR, bool FUSED>
__global__ void __launch_bounds__(256) gemm_f32_kernel(GemmF32Dev p) {
  constexpr int BM = 16 * TM, BN = 16 * TN;
  __shared__ f32x4 part_sum[kKParts][TM * TN][64];
  __shared__ int32_t list[FUSED ? kSelMaxTokensF32 : 1], wave_tot[4];
  int m;
  if constexpr (FUSED)
    m = derive_rows_f32(p, list, wave_tot);
  else
    m = p.m_dev ? *p.m_dev : p.m_max;
  const int m0 = blockIdx.x * BM, n0 = blockIdx.y * BN;
  if (m0 >= m) return;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l16 = lane & 15, kq = lane >> 4;

  long tok[TM];
  const float* asrc[TM];
  const float* bsrc[TN];
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    int row = m0 + i * 16 + l16;
    row = row < m ? row : m - 1;
    tok[i] = FUSED ? (long)list[row] : (p.idx ? (long)p.idx[row] : (long)row);
    asrc[i] = p.a + tok[i] * p.lda + kq * 4;
  }
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    int col = n0 + j * 16 + l16;
    col = col < p.n ? col : p.n - 1;
    bsrc[j] = p.wt + (long)col * p.k + kq * 4;
  }

  const int steps = p.k / (16 * kKParts);  // per quarter
  // the sum over the wave's quarter, chunks of UNR steps whose loads are all in flight at once
  f32x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int kbase = wave * steps * 16;
  for (int s = 0; s < steps; s += UNR) {
    f32x4 fa[UNR][TM], fb[UNR][TN];
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      const int k0 = kbase + (s + u < steps ? s + u : steps - 1) * 16;
#pragma unroll
      for (int i = 0; i < TM; ++i) fa[u][i] = *reinterpret_cast<const f32x4*>(asrc[i] + k0);
#pragma unroll
      for (int j = 0; j < TN; ++j) fb[u][j] = *reinterpret_cast<const f32x4*>(bsrc[j] + k0);
    }
    if constexpr (UNR > 1) {
      // (all in flight: the compiler moved a load behind the break in front of its use, 28 registers for 60, and waited for each;
      // a KV+O step of 1 x 256 tokens of hidden 4096 455 -> 444 us, of 1 x 1024 of 1024 178 -> 174)
#pragma unroll
      for (int u = 0; u < UNR; ++u) {
#pragma unroll
        for (int i = 0; i < TM; ++i) asm volatile("" : "+v"(fa[u][i]));
#pragma unroll
        for (int j = 0; j < TN; ++j) asm volatile("" : "+v"(fb[u][j]));
      }
    }
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      if (s + u >= steps) break;  // (uniform)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fb[u][j][e], fa[u][i][e], acc[i][j], 0, 0, 0);
    }
  }

  // acc[i][j][e]: row 16 i + l16, column 16 j + 4 kq + e of the tile
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) part_sum[wave][i * TN + j][lane] = acc[i][j];
  __syncthreads();
#pragma unroll
  for (int t = 0; t < TM * TN; ++t) {
    if (t % 4 != wave) continue;
    const int i = t / TN, j = t % TN;
    f32x4 v = part_sum[0][t][lane];
#pragma unroll
    for (int w = 1; w < kKParts; ++w) v += part_sum[w][t][lane];
    const int row = m0 + i * 16 + l16, col = n0 + j * 16 + kq * 4;
    if (row < m && col < p.n) store4_f32(p, tok[i], col, v);
  }
}

template <int TM, int TN, int UNR>
hipError_t launch_shape(const GemmF32Dev& p, hipStream_t s) {
  constexpr int BM = 16 * TM, BN = 16 * TN;
  const int tm = (p.m_max + BM - 1) / BM, tn = (p.n + BN - 1) / BN;
  if (tm == 0 || tn == 0) return hipSuccess;
  if (p.sel_mask)
    hipLaunchKernelGGL((gemm_f32_kernel<TM, TN, UNR, true>), dim3(tm, tn), dim3(256), 0, s, p);
  else
    hipLaunchKernelGGL((gemm_f32_kernel<TM, TN, UNR, false>), dim3(tm, tn), dim3(256), 0, s, p);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_gemm_f32(const GemmArgs& g, hipStream_t s) {
  GemmF32Dev p;
  p.a = static_cast<const float*>(g.a);
  p.wt = static_cast<const float*>(g.wt);
  p.idx = g.idx;
  p.m_dev = g.m_dev;
  p.c0 = static_cast<float*>(g.c[0]);
  p.c1 = static_cast<float*>(g.c[1]);
  p.c2 = static_cast<float*>(g.c[2]);
  p.c32 = g.c32;
  p.lda = g.lda;
  p.n = g.n;
  p.k = g.k;
  p.m_max = g.m_max;
  p.ldc = g.ldc;
  p.seg_n = g.seg_n;
  p.c32_cols = g.c32_cols;
  p.rope = g.rope;
  p.rope_cols = g.rope_cols;
  p.rope_dh = g.rope_dh;
  p.rope_seq = g.rope_seq;
  p.sel_mask = g.sel_mask;
  p.sel_batch = g.sel_batch;
  p.sel_seq = g.sel_seq;
  p.sel_idx_out = g.sel_idx_out;
  p.sel_idx_out2 = g.sel_idx_out2;
  p.sel_off_out = g.sel_off_out;
  p.sel_count_out = g.sel_count_out;
  if (p.sel_mask && (long)g.sel_batch * g.sel_seq > kSelMaxTokensF32) return hipErrorInvalidValue;
  // The largest tile that gives most of the chip's 256 CUs a workgroup.  Measured (us; before: 64 x 64
  // tiles through LDS): 1024 x 12288 x 4096 1325 -> 880, 1024 x 2048 x 2048 141 -> 80 and
  // 514 x 3072 x 1024 74 -> 46, 32 x 126464 x 4096 920 -> 691, 205 refreshed of 1024 rows x 12288 x 4096 1095 ->
  // 925 (64 x 64), 64 x 4096 x 4096 235 -> 43 (32 x 32; 64 with 16 x 16, 84 with 64 x 64).
  auto tiles = [&](int b) { return (long)((g.m_max + b - 1) / b) * ((g.n + b - 1) / b); };
  constexpr long kFill = 192;
  if (tiles(64) >= kFill) return launch_shape<4, 4, 1>(p, s);
  if (tiles(32) >= kFill) return launch_shape<2, 2, 4>(p, s);
  return launch_shape<1, 1, 4>(p, s);
}

}  // namespace dare
