// Device helpers shared by the row-wise kernels: a wavefront holds one row of D values in registers, as up to MAXC
// 16-byte chunks per lane (chunk lane + 64 i), converted to fp32.
#pragma once
#include "bsr_internal.h"

namespace bsr {

constexpr int WAVE = 64;
constexpr int ROW_MAX = 2048;       // longest row these kernels take

template <typename T> struct Chunk { static constexpr int V = 16 / sizeof(T); typedef T vec __attribute__((ext_vector_type(16 / sizeof(T)))); };

// Sums and maxima over a wavefront, in every lane; the pairs are those of an exchange with lane ^ 32, ^ 16, ... ^ 1.  They stay on the vector
// unit: gfx950 swaps half waves and rows of 16 lanes, and once lanes 8 (then 4) apart hold the same value, a rotation by 8 (by 4)
// within a row is the exchange with lane ^ 8 (lane ^ 4).  A row kernel waits for two such sums one after the other, and through LDS (ds_bpermute)
// each of the six steps took its latency.  With the loads below: the LayerNorms of a ViT-B step of 32 images 123 -> 115 us forward and 62 -> 60
// backward, of DeiT-S 93 -> 88 and 48 -> 44, whole steps 2280 -> 2245 and 1275 -> 1254.
template <int CTRL> __device__ __forceinline__ float dpp_move(float v) {
  return __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(v), CTRL, 0xf, 0xf, true));
}
template <class Op> __device__ __forceinline__ float halves_all(float v, Op op) {      // of lanes l and l ^ 32
  const auto halves = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return op(__uint_as_float(halves[0]), __uint_as_float(halves[1]));
}
template <class Op> __device__ __forceinline__ float wave_all(float v, Op op) {
  v = halves_all(v, op);
  const auto rows = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = op(__uint_as_float(rows[0]), __uint_as_float(rows[1]));
  v = op(v, dpp_move<0x128>(v));       // row_ror:8
  v = op(v, dpp_move<0x124>(v));       // row_ror:4
  v = op(v, dpp_move<0x4E>(v));        // quad_perm:[2,3,0,1]
  return op(v, dpp_move<0xB1>(v));     // quad_perm:[1,0,3,2]
}
__device__ inline float half_sum(float v) { return halves_all(v, [](float a, float b) { return a + b; }); }
__device__ inline float half_max(float v) { return halves_all(v, [](float a, float b) { return fmaxf(a, b); }); }
__device__ inline float half_other(float v) {                    // the value of lane ^ 32
  const auto halves = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(threadIdx.x & 32 ? halves[0] : halves[1]);
}
__device__ inline float wave_sum(float v) { return wave_all(v, [](float a, float b) { return a + b; }); }
__device__ inline float wave_max(float v) { return wave_all(v, [](float a, float b) { return fmaxf(a, b); }); }
// over each eight lanes: lane ^ 1, ^ 2, ^ 4 (the quads hold one value by then, so mirroring the eight lanes is that exchange)
__device__ inline float eight_sum(float v) {
  v += dpp_move<0xB1>(v);
  v += dpp_move<0x4E>(v);
  return v + dpp_move<0x141>(v);       // row_half_mirror
}

// V consecutive fp32 parameters
template <int V> __device__ __forceinline__ void load_params(const float* p, float (&o)[V]) {
#pragma unroll
  for (int q = 0; q < V / 4; ++q) {
    const float4 t = *(const float4*)(p + 4 * q);
    o[4 * q] = t.x; o[4 * q + 1] = t.y; o[4 * q + 2] = t.z; o[4 * q + 3] = t.w;
  }
}

// The row at x in v as fp32, zero past its end.  No branch around the loads: a lane past the end reads the last chunk again (with a branch
// each, the loads of a row waited for one another).
template <typename T, int MAXC>
__device__ __forceinline__ void load_row(const T* x, int nch, int lane, typename Chunk<T>::vec (&raw)[MAXC], float (&v)[MAXC][Chunk<T>::V]) {
#pragma unroll
  for (int i = 0; i < MAXC; ++i) raw[i] = *(const typename Chunk<T>::vec*)(x + min(lane + i * WAVE, nch - 1) * Chunk<T>::V);
#pragma unroll
  for (int i = 0; i < MAXC; ++i)
#pragma unroll
    for (int e = 0; e < Chunk<T>::V; ++e) v[i][e] = lane + i * WAVE < nch ? (float)raw[i][e] : 0.f;
}

// LayerNorm of the row in v (zero past its end; fp32 statistics, mean first, then the biased variance): y = (x - mean) rstd gamma + beta.
// gamma and beta are asked for ahead of the sums where they fit: behind the sums, and behind the stores of mean and rstd, a row
// waits for memory twice.
template <typename T, int MAXC, bool FITS = (MAXC <= 2)> struct RowParams {
  static constexpr bool AHEAD = FITS;
  float g[AHEAD ? MAXC : 1][Chunk<T>::V], b[AHEAD ? MAXC : 1][Chunk<T>::V];
  __device__ __forceinline__ void load(const float* __restrict__ gamma, const float* __restrict__ beta, int c, int i) {
    load_params<Chunk<T>::V>(gamma + c * Chunk<T>::V, g[i]);
    load_params<Chunk<T>::V>(beta + c * Chunk<T>::V, b[i]);
  }
  __device__ __forceinline__ void ahead(const float* __restrict__ gamma, const float* __restrict__ beta, int nch, int lane) {
    if constexpr (AHEAD)
#pragma unroll
      for (int i = 0; i < MAXC; ++i) load(gamma, beta, min(lane + i * WAVE, nch - 1), i);
  }
};
template <typename T, int MAXC, bool AHEAD>
__device__ __forceinline__ void layernorm_row(const float (&v)[MAXC][Chunk<T>::V], RowParams<T, MAXC, AHEAD>& par, int D, int lane,
                                              const float* __restrict__ gamma, const float* __restrict__ beta, float eps, T* __restrict__ y,
                                              float* mean, float* rstd) {
  constexpr int V = Chunk<T>::V;
  const int nch = D / V;
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < MAXC; ++i)
#pragma unroll
    for (int e = 0; e < V; ++e) s += v[i][e];
  const float mu = wave_sum(s) / (float)D;
  float q = 0.f;
#pragma unroll
  for (int i = 0; i < MAXC; ++i)
#pragma unroll
    for (int e = 0; e < V; ++e) { const float d0 = lane + i * WAVE < nch ? v[i][e] - mu : 0.f; q += d0 * d0; }
  const float rs = rsqrtf(wave_sum(q) / (float)D + eps);
  if (lane == 0) {
    if (mean) *mean = mu;
    if (rstd) *rstd = rs;
  }
#pragma unroll
  for (int i = 0; i < MAXC; ++i) {
    const int c = lane + i * WAVE;
    if (c < nch) {
      if constexpr (!AHEAD) par.load(gamma, beta, c, 0);
      typename Chunk<T>::vec o;
#pragma unroll
      for (int e = 0; e < V; ++e) o[e] = (T)((v[i][e] - mu) * rs * par.g[AHEAD ? i : 0][e] + par.b[AHEAD ? i : 0][e]);
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
