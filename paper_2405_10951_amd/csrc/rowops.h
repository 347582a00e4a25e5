// Device helpers shared by the row-wise kernels: a wavefront holds one row of D values in registers, as up to MAXC
// 16-byte chunks per lane (chunk lane + 64 i), converted to fp32.
#pragma once
#include "bsr_internal.h"

namespace bsr {

constexpr int WAVE = 64;
constexpr int ROW_MAX = 2048;       // longest row these kernels take

template <typename T> struct Chunk { static constexpr int V = 16 / sizeof(T); typedef T vec __attribute__((ext_vector_type(16 / sizeof(T)))); };

__device__ inline float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, WAVE);
  return v;
}
__device__ inline float wave_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, WAVE));
  return v;
}

// V consecutive fp32 parameters
template <int V> __device__ __forceinline__ void load_params(const float* p, float (&o)[V]) {
#pragma unroll
  for (int q = 0; q < V / 4; ++q) {
    const float4 t = *(const float4*)(p + 4 * q);
    o[4 * q] = t.x; o[4 * q + 1] = t.y; o[4 * q + 2] = t.z; o[4 * q + 3] = t.w;
  }
}

// LayerNorm of the row in v (fp32 statistics, mean first, then the biased variance): y = (x - mean) rstd gamma + beta
template <typename T, int MAXC>
__device__ __forceinline__ void layernorm_row(const float (&v)[MAXC][Chunk<T>::V], int D, int lane, const float* __restrict__ gamma,
                                              const float* __restrict__ beta, float eps, T* __restrict__ y, float* mean, float* rstd) {
  constexpr int V = Chunk<T>::V;
  const int nch = D / V;
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < MAXC; ++i)
    if (lane + i * WAVE < nch)
#pragma unroll
      for (int e = 0; e < V; ++e) s += v[i][e];
  const float mu = wave_sum(s) / (float)D;
  float q = 0.f;
#pragma unroll
  for (int i = 0; i < MAXC; ++i)
    if (lane + i * WAVE < nch)
#pragma unroll
      for (int e = 0; e < V; ++e) { const float d0 = v[i][e] - mu; q += d0 * d0; }
  const float rs = rsqrtf(wave_sum(q) / (float)D + eps);
  if (lane == 0) {
    if (mean) *mean = mu;
    if (rstd) *rstd = rs;
  }
#pragma unroll
  for (int i = 0; i < MAXC; ++i) {
    const int c = lane + i * WAVE;
    if (c < nch) {
      float gg[V], bb[V];
      load_params<V>(gamma + c * V, gg);
      load_params<V>(beta + c * V, bb);
      typename Chunk<T>::vec o;
#pragma unroll
      for (int e = 0; e < V; ++e) o[e] = (T)((v[i][e] - mu) * rs * gg[e] + bb[e]);
      *(typename Chunk<T>::vec*)(y + c * V) = o;
    }
  }
}

// f(IC<MAXC>) for the chunk count of rows of D elements of T (D a multiple of the chunk length, at most ROW_MAX)
template <int V> struct RowC { static constexpr int value = V; };
template <typename T, class F> inline bool with_row_chunks(int D, F&& f) {
  constexpr int V = Chunk<T>::V;
  if (D % V || D > ROW_MAX) return false;
  const int per_lane = (D / V + WAVE - 1) / WAVE;
  if (per_lane <= 1) f(RowC<1>{});
  else if (per_lane <= 2) f(RowC<2>{});
  else if (per_lane <= 4) f(RowC<4>{});
  else f(RowC<8>{});
  return true;
}

}  // namespace bsr
