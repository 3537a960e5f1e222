// fp32 path of the selected-row bidirectional attention (App. E.2; Alg. 1 line 10; Alg. 2
// line 8) on v_mfma_f32_16x16x4_f32.
//
// A workgroup serves 16 query rows of one (sequence, head); its four waves take every fourth
// tile of 32 keys (16 where a head has 128 channels, whose tiles take twice the registers).  Transposed logits S^T = K Q^T (key fragment first): lane L holds query
// L & 15 and four neighbouring keys per 16, which is the operand layout of the probabilities in
// O^T = V^T P^T, so they never leave the lane.  K, V and Q go from global memory straight into
// registers (a fragment is used by one wave only), all loads of a tile in flight at once.  The
// key-waves are merged in wave order through LDS.
//
// What bounds it: at the short sequences of the fp32 configurations the latency of one
// workgroup.  128 keys, 26 queries, 4 heads of 64: 14.2 -> 6.4 us against one wave per query that read
// a key row per lane and walked the values key by key; -> 5.4 us with the first tile requested ahead of the reads that lead
// to the queries and the loads kept together (the scheduler had spread them over the MFMAs of their uses, a wait each).  Whole KV+O
// steps by the latter: 1 x 128 tokens of hidden 256 20.6 -> 19.2 us, 8 x 1024 of 256 137 -> 114, with 4 heads of 128 241 -> 219,
// 4 x 1024 of 4096 3352 -> 3154.
#include "dare_common.h"

namespace dare {
namespace {

constexpr int kWaves = 4;  // key-waves

struct AttnF32Dev {
  const float* q;
  const float* k;
  const float* v;
  float* out;
  const int32_t* idx;
  const int32_t* sel_off;
  int seq, d;
  float scale;
};

// over the four lanes that hold the same query
__device__ __forceinline__ float query_max(float v) {
  v = fmaxf(v, __shfl_xor(v, 16, 64));
  return fmaxf(v, __shfl_xor(v, 32, 64));
}
__device__ __forceinline__ float query_sum(float v) {
  v += __shfl_xor(v, 16, 64);
  return v + __shfl_xor(v, 32, 64);
}

template <int DH>
__global__ void __launch_bounds__(kWaves * 64) attn_f32_kernel(AttnF32Dev p) {
  constexpr int C = DH / 16;  // 16-channel tiles
  constexpr int kTiles = DH == 64 ? 2 : 1;  // 16-key tiles per wave and step
  __shared__ f32x4 o_part[kWaves][C][64];
  __shared__ float m_part[kWaves][16], l_part[kWaves][16];
  const int b = blockIdx.z, h = blockIdx.y;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l16 = lane & 15, kq = lane >> 4;
  const int T = p.seq;
  int cnt, off;
  if (p.idx) {
    off = p.sel_off[b];
    cnt = p.sel_off[b + 1] - off;
  } else {
    off = b * T;
    cnt = T;
  }
  if ((int)blockIdx.x * 16 >= cnt) return;  // uniform for the workgroup
  const float* kbase = p.k + (long)b * T * p.d + h * DH;
  const float* vbase = p.v + (long)b * T * p.d + h * DH;
  f32x4 kf[kTiles][C];
  float vf[kTiles][4][C];
  // (the scheduler moves loads back to their uses, one wait after the other, unless it is kept from it)
  auto load_tiles = [&](int key0) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < kTiles; ++t) {
      int key = key0 + t * 16 + l16;
      key = key < T ? key : T - 1;
#pragma unroll
      for (int c = 0; c < C; ++c) kf[t][c] = *reinterpret_cast<const f32x4*>(kbase + (long)key * p.d + c * 16 + kq * 4);
    }
#pragma unroll
    for (int t = 0; t < kTiles; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int key = key0 + t * 16 + kq * 4 + e;
        const float* vr = vbase + (long)(key < T ? key : T - 1) * p.d + l16;
#pragma unroll
        for (int c = 0; c < C; ++c) vf[t][e][c] = vr[c * 16];
      }
    __builtin_amdgcn_sched_barrier(0);
  };
  load_tiles(wave * (16 * kTiles));  // (under the two dependent reads that lead to the queries)

  const int j = blockIdx.x * 16 + l16;
  const bool valid = j < cnt;
  const int jc = valid ? j : cnt - 1;
  const long tok = p.idx ? (long)p.idx[off + jc] : (long)(off + jc);

  // channels 16 c + 4 kq .. + 3 of the lane's query
  f32x4 qf[C];
#pragma unroll
  for (int c = 0; c < C; ++c) qf[c] = *reinterpret_cast<const f32x4*>(p.q + tok * p.d + h * DH + c * 16 + kq * 4);

  f32x4 acc[C];
#pragma unroll
  for (int c = 0; c < C; ++c) acc[c] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m_run = -INFINITY, l_run = 0.f;

  constexpr int kStep = kWaves * 16 * kTiles;
  for (int key0 = wave * (16 * kTiles); key0 < T; key0 += kStep) {
    // z[t][e]: logit of key key0 + 16 t + 4 kq + e
    f32x4 z[kTiles];
    float m_loc = -INFINITY;
#pragma unroll
    for (int t = 0; t < kTiles; ++t) {
      z[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int c = 0; c < C; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e) z[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[t][c][e], qf[c][e], z[t], 0, 0, 0);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        z[t][e] = key0 + t * 16 + kq * 4 + e < T ? z[t][e] * p.scale : -INFINITY;
        m_loc = fmaxf(m_loc, z[t][e]);
      }
    }
    const float m_new = fmaxf(m_run, query_max(m_loc));
    // (a tile whose logits are all -inf adds nothing; -inf - -inf would be NaN)
    const float m_ref = m_new == -INFINITY ? 0.f : m_new;
    const float alpha = expf(m_run - m_ref);
    m_run = m_new;
    l_run *= alpha;
#pragma unroll
    for (int c = 0; c < C; ++c) acc[c] *= alpha;
#pragma unroll
    for (int t = 0; t < kTiles; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const bool live = key0 + t * 16 + kq * 4 + e < T;
        const float pr = expf(z[t][e] - m_ref);
        l_run += pr;
#pragma unroll
        for (int c = 0; c < C; ++c)
          acc[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(live ? vf[t][e][c] : 0.f, pr, acc[c], 0, 0, 0);
      }
    if (key0 + kStep < T) load_tiles(key0 + kStep);
  }
  l_run = query_sum(l_run);
  if (kq == 0) {
    m_part[wave][l16] = m_run;
    l_part[wave][l16] = l_run;
  }
#pragma unroll
  for (int c = 0; c < C; ++c) o_part[wave][c][lane] = acc[c];
  __syncthreads();
  float m_all = m_part[0][l16], l_all = 0.f, f[kWaves];
#pragma unroll
  for (int w = 1; w < kWaves; ++w) m_all = fmaxf(m_all, m_part[w][l16]);
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    f[w] = expf(m_part[w][l16] - m_all);
    l_all += l_part[w][l16] * f[w];
  }
  if (!valid) return;
  const float inv = 1.0f / l_all;
  // acc[c][e]: channel 16 c + 4 kq + e of the lane's query
  for (int c = wave; c < C; c += kWaves) {
    f32x4 o = o_part[0][c][lane] * f[0];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) o += o_part[w][c][lane] * f[w];
    *reinterpret_cast<f32x4*>(p.out + tok * p.d + h * DH + c * 16 + kq * 4) = o * inv;
  }
}

}  // namespace

hipError_t launch_attn_f32(const AttnArgs& a, hipStream_t s) {
  AttnF32Dev p;
  p.q = static_cast<const float*>(a.q);
  p.k = static_cast<const float*>(a.k);
  p.v = static_cast<const float*>(a.v);
  p.out = static_cast<float*>(a.out);
  p.idx = a.idx;
  p.sel_off = a.sel_off;
  p.seq = a.seq;
  p.d = a.n_heads * a.head_dim;
  p.scale = 1.0f / sqrtf((float)a.head_dim);
  dim3 grid((a.seq + 15) / 16, a.n_heads, a.batch);
  if (a.head_dim == 128)
    hipLaunchKernelGGL(attn_f32_kernel<128>, grid, dim3(kWaves * 64), 0, s, p);
  else if (a.head_dim == 64)
    hipLaunchKernelGGL(attn_f32_kernel<64>, grid, dim3(kWaves * 64), 0, s, p);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace dare
