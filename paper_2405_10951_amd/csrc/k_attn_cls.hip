// Attention of the class token alone (query 0 of every image and head), forward and backward: all that the last block of
// a classifier needs, since the head reads nothing else of its output.  fp32 arithmetic on fp32 or bf16 storage.
//
// Bound by memory: forward reads K and V once, backward reads K twice (for the scores and for dQ) and V once and writes dQ, dK
// and dV once, each 16 bytes per lane with eight lanes on a row of 64 bf16 values.  One workgroup per (image, head).
#include "rowops.h"

namespace bsr {

namespace {

constexpr int MAX_T = 1024, NT = 256, NW = NT / WAVE, GL = 8, NG = NT / GL;   // eight lanes per key, NG keys at a time

__device__ inline float block_sum(float v, float* red) {
  v = wave_sum(v);
  __syncthreads();
  if (threadIdx.x % WAVE == 0) red[threadIdx.x / WAVE] = v;
  __syncthreads();
  return (red[0] + red[1]) + (red[2] + red[3]);
}
__device__ inline float block_max(float v, float* red) {
  v = wave_max(v);
  __syncthreads();
  if (threadIdx.x % WAVE == 0) red[threadIdx.x / WAVE] = v;
  __syncthreads();
  return fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
}
// adds acc (this lane's chunk c of a row, one partial per key group) over the NG groups, in group order; valid in group 0
template <int V> __device__ __forceinline__ void groups_sum(float (&acc)[V], float* red, int grp, int gl) {
  __syncthreads();
#pragma unroll
  for (int e = 0; e < V; ++e) red[(grp * GL + gl) * V + e] = acc[e];
  __syncthreads();
  if (grp != 0) return;
  for (int g = 1; g < NG; ++g)
#pragma unroll
    for (int e = 0; e < V; ++e) acc[e] += red[(g * GL + gl) * V + e];
}

// out [B, H d] (one row per image), lse [B, H]
template <typename T>
__global__ __launch_bounds__(NT) void attn_cls_fwd_kernel(const T* __restrict__ qkv, int T_, int H, int d, T* __restrict__ out,
                                                          float* __restrict__ lse) {
  constexpr int V = Chunk<T>::V;
  typedef typename Chunk<T>::vec vec;
  __shared__ float p[MAX_T], red[NT * V], rs4[NW];
  const int b = blockIdx.x / H, h = blockIdx.x % H, D = H * d, nch = d / V, gl = threadIdx.x % GL, grp = threadIdx.x / GL;
  const T* base = qkv + (int64_t)b * T_ * 3 * D + h * d;
  const float scale = rsqrtf((float)d);
  float mx = -INFINITY;
  for (int j = grp; j < T_; j += NG) {
    float s = 0.f;
    for (int c = gl; c < nch; c += GL) {
      const vec q = *(const vec*)(base + c * V), k = *(const vec*)(base + (int64_t)j * 3 * D + D + c * V);
#pragma unroll
      for (int e = 0; e < V; ++e) s = fmaf((float)q[e], (float)k[e], s);
    }
    s = eight_sum(s) * scale;
    if (gl == 0) p[j] = s;
    mx = fmaxf(mx, s);
  }
  mx = block_max(mx, rs4);                 // (the barrier in it also publishes p)
  float sum = 0.f;
  for (int j = threadIdx.x; j < T_; j += NT) {
    const float e = expf(p[j] - mx);
    p[j] = e;
    sum += e;
  }
  sum = block_sum(sum, rs4);
  const float inv = 1.0f / sum;
  if (threadIdx.x == 0) lse[blockIdx.x] = mx + logf(sum);
  for (int c0 = 0; c0 < nch; c0 += GL) {   // (uniform trip count: the sum over groups has barriers)
    const int c = c0 + gl;
    float acc[V];
#pragma unroll
    for (int e = 0; e < V; ++e) acc[e] = 0.f;
    if (c < nch)
#pragma unroll 4
      for (int j = grp; j < T_; j += NG) {
        const vec v = *(const vec*)(base + (int64_t)j * 3 * D + 2 * D + c * V);
        const float pj = p[j];
#pragma unroll
        for (int e = 0; e < V; ++e) acc[e] = fmaf(pj, (float)v[e], acc[e]);
      }
    groups_sum<V>(acc, red, grp, gl);
    if (grp == 0 && c < nch) {
      vec o;
#pragma unroll
      for (int e = 0; e < V; ++e) o[e] = (T)(acc[e] * inv);
      *(vec*)(out + (int64_t)b * D + h * d + c * V) = o;
    }
  }
}

// Eq. 3, 5 with a gradient dout [B, H d] at query 0 only: P_j = exp(s_j - lse), dP_j = dO . v_j, delta = sum_j P_j dP_j (the
// stored output is rounded, so not dO . O), dS_j = P_j (dP_j - delta) / sqrt d; dK_j = dS_j q, dV_j = P_j dO,
// dQ_0 = sum_j dS_j k_j, dQ_j = 0.
template <typename T>
__global__ __launch_bounds__(NT) void attn_cls_bwd_kernel(const T* __restrict__ qkv, const T* __restrict__ dout,
                                                          const float* __restrict__ lse, int T_, int H, int d, T* __restrict__ dqkv) {
  constexpr int V = Chunk<T>::V;
  typedef typename Chunk<T>::vec vec;
  __shared__ float p[MAX_T], dp[MAX_T], red[NT * V], rs4[NW];
  const int b = blockIdx.x / H, h = blockIdx.x % H, D = H * d, nch = d / V, gl = threadIdx.x % GL, grp = threadIdx.x / GL;
  const T* base = qkv + (int64_t)b * T_ * 3 * D + h * d;
  T* dbase = dqkv + (int64_t)b * T_ * 3 * D + h * d;
  const T* dorow = dout + (int64_t)b * D + h * d;
  const float scale = rsqrtf((float)d), l = lse[blockIdx.x];
  float delta = 0.f;
  for (int j = grp; j < T_; j += NG) {
    const T* kr = base + (int64_t)j * 3 * D + D;
    float s = 0.f, t = 0.f;
    for (int c = gl; c < nch; c += GL) {
      const vec q = *(const vec*)(base + c * V), k = *(const vec*)(kr + c * V), v = *(const vec*)(kr + D + c * V), g = *(const vec*)(dorow + c * V);
#pragma unroll
      for (int e = 0; e < V; ++e) { s = fmaf((float)q[e], (float)k[e], s); t = fmaf((float)g[e], (float)v[e], t); }
    }
    const float pj = expf(eight_sum(s) * scale - l), dpj = eight_sum(t);
    if (gl == 0) { p[j] = pj; dp[j] = dpj; delta = fmaf(pj, dpj, delta); }
  }
  delta = block_sum(delta, rs4);           // (the barriers in it also publish p and dp)
  for (int j = grp; j < T_; j += NG) {
    T* dr = dbase + (int64_t)j * 3 * D;
    const float pj = p[j], dsj = pj * (dp[j] - delta) * scale;
    for (int c = gl; c < nch; c += GL) {
      const vec q = *(const vec*)(base + c * V), g = *(const vec*)(dorow + c * V);
      vec dk, dv;
#pragma unroll
      for (int e = 0; e < V; ++e) { dk[e] = (T)(dsj * (float)q[e]); dv[e] = (T)(pj * (float)g[e]); }
      if (j > 0) *(vec*)(dr + c * V) = (vec)(T)0.f;
      *(vec*)(dr + D + c * V) = dk;
      *(vec*)(dr + 2 * D + c * V) = dv;
    }
  }
  for (int c0 = 0; c0 < nch; c0 += GL) {
    const int c = c0 + gl;
    float acc[V];
#pragma unroll
    for (int e = 0; e < V; ++e) acc[e] = 0.f;
    if (c < nch)
#pragma unroll 4
      for (int j = grp; j < T_; j += NG) {
        const vec k = *(const vec*)(base + (int64_t)j * 3 * D + D + c * V);
        const float w = p[j] * (dp[j] - delta) * scale;
#pragma unroll
        for (int e = 0; e < V; ++e) acc[e] = fmaf(w, (float)k[e], acc[e]);
      }
    groups_sum<V>(acc, red, grp, gl);
    if (grp == 0 && c < nch) {
      vec o;
#pragma unroll
      for (int e = 0; e < V; ++e) o[e] = (T)acc[e];
      *(vec*)(dbase + c * V) = o;
    }
  }
}

}  // namespace

bool attn_cls_supported(int T, int d, bool f32) { return T >= 1 && T <= MAX_T && d % (f32 ? 4 : 8) == 0; }

void attn_cls_fwd(const void* qkv, int B, int T, int H, int d, bool f32, void* out, float* lse, hipStream_t s) {
  if (f32) attn_cls_fwd_kernel<float><<<B * H, NT, 0, s>>>((const float*)qkv, T, H, d, (float*)out, lse);
  else attn_cls_fwd_kernel<bf16><<<B * H, NT, 0, s>>>((const bf16*)qkv, T, H, d, (bf16*)out, lse);
}

void attn_cls_bwd(const void* qkv, const void* dout, const float* lse, int B, int T, int H, int d, bool f32,
                  void* dqkv, hipStream_t s) {
  if (f32) attn_cls_bwd_kernel<float><<<B * H, NT, 0, s>>>((const float*)qkv, (const float*)dout, lse, T, H, d, (float*)dqkv);
  else attn_cls_bwd_kernel<bf16><<<B * H, NT, 0, s>>>((const bf16*)qkv, (const bf16*)dout, lse, T, H, d, (bf16*)dqkv);
}

}  // namespace bsr
