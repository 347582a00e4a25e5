// LayerNorm forward and backward.  One wavefront per row, the row read once with 16-byte loads and kept in registers
// (rows of whole 16-byte chunks up to 2048 long; others go through the generic kernels).  Bound by memory; reductions
// over rows are two-pass with a fixed order, so results are bit-reproducible.
#include <algorithm>

#include "rowops.h"

namespace bsr {

namespace {

constexpr int COLSUM_R = 64;      // row chunks of the generic column reduction
constexpr int FINAL_WAVES = 16;

template <typename T, int MAXC>
__global__ __launch_bounds__(256) void ln_fwd_kernel(const T* __restrict__ x, int64_t M, int D, const float* __restrict__ gamma,
                                                     const float* __restrict__ beta, float eps, T* __restrict__ y,
                                                     float* __restrict__ mean, float* __restrict__ rstd) {
  const int lane = threadIdx.x % WAVE;
  const int64_t m = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
  if (m >= M) return;
  typename Chunk<T>::vec raw[MAXC];
  float v[MAXC][Chunk<T>::V];
  load_row<T, MAXC>(x + m * D, D / Chunk<T>::V, lane, raw, v);
  RowParams<T, MAXC> par;
  par.ahead(gamma, beta, D / Chunk<T>::V, lane);
  layernorm_row(v, par, D, lane, gamma, beta, eps, y + m * D, mean ? mean + m : nullptr, rstd ? rstd + m : nullptr);
}

// any row length
template <typename T>
__global__ __launch_bounds__(256) void ln_fwd_any_kernel(const T* __restrict__ x, int64_t M, int D, const float* __restrict__ gamma,
                                                         const float* __restrict__ beta, float eps, T* __restrict__ y,
                                                         float* __restrict__ mean, float* __restrict__ rstd) {
  const int lane = threadIdx.x % WAVE;
  const int64_t m = (int64_t)blockIdx.x * 4 + threadIdx.x / WAVE;
  if (m >= M) return;
  const T* xr = x + m * D;
  float s = 0.f;
  for (int j = lane; j < D; j += WAVE) s += (float)xr[j];
  const float mu = wave_sum(s) / (float)D;
  float v = 0.f;
  for (int j = lane; j < D; j += WAVE) {
    const float c = (float)xr[j] - mu;
    v += c * c;
  }
  const float rs = rsqrtf(wave_sum(v) / (float)D + eps);
  if (lane == 0) {
    if (mean) mean[m] = mu;
    if (rstd) rstd[m] = rs;
  }
  for (int j = lane; j < D; j += WAVE) y[m * D + j] = (T)(((float)xr[j] - mu) * rs * gamma[j] + beta[j]);
}

// the residual row of row m, null where it has none
template <typename T> __device__ inline const T* res_row(const LnRows<T>& r, int64_t m, int D) {
  if (!r.res) return nullptr;
  if (r.res_period == 0) return r.res + m * D;
  return m % r.res_period == 0 ? r.res + m / r.res_period * D : nullptr;
}

// Where the gradient of a row goes (LnRows); the rows of the tokens dropped since the row before it, and behind an image's last one, are cleared
// by the wavefront that has the row: every row of dx is written exactly once, without a search.
struct RowPlace {
  unsigned image = 0;
  int token = 0, before = 0;      // places of this row and of the one before it (-1: none)
  bool last = false;
  __device__ __forceinline__ void find(const LnScatter& sc, int64_t m) {       // (row counts fit 31 bits)
    const unsigned n = (unsigned)sc.k + 1u;
    image = (unsigned)m / n;
    const int i = (int)((unsigned)m % n);
    const int32_t* idx = sc.idx + (int64_t)image * sc.k;
    token = i == 0 ? 0 : 1 + idx[i - 1];
    before = i == 0 ? -1 : i == 1 ? 0 : 1 + idx[i - 2];
    last = i == sc.k;
  }
  template <typename T> __device__ __forceinline__ T* row(const LnRows<T>& r, int D, int lane) const {
    T* img = r.dx + (int64_t)image * r.sc.T * D;
    auto clear = [&](int t0, int t1) {
      uint4* z = (uint4*)(img + (int64_t)t0 * D);
      for (int j = lane; j < (t1 - t0) * (D * (int)sizeof(T) / 16); j += WAVE) z[j] = make_uint4(0u, 0u, 0u, 0u);
    };
    clear(before + 1, token);
    if (last) clear(token + 1, r.sc.T);
    return img + (int64_t)token * D;
  }
};

// dx = res + rstd * (g - mean(g) - xhat * mean(g * xhat)),  g = dy * gamma; any row length
template <typename T>
__global__ __launch_bounds__(256) void ln_bwd_dx_any_kernel(const T* __restrict__ dy, LnRows<T> r, int64_t M, int D,
                                                            const float* __restrict__ mean, const float* __restrict__ rstd,
                                                            const float* __restrict__ gamma) {
  const int lane = threadIdx.x % WAVE;
  const int64_t m = (int64_t)blockIdx.x * (blockDim.x / WAVE) + threadIdx.x / WAVE;
  if (m >= M) return;
  const float mu = mean[m], rs = rstd[m];
  const T* dyr = dy + m * D;
  const T* xr = r.x + m * D;
  const T* rr = res_row(r, m, D);
  float s1 = 0.f, s2 = 0.f;
  for (int j = lane; j < D; j += WAVE) {
    const float g = (float)dyr[j] * gamma[j];
    s1 += g;
    s2 += g * ((float)xr[j] - mu) * rs;
  }
  const float m1 = wave_sum(s1) / (float)D, m2 = wave_sum(s2) / (float)D;
  for (int j = lane; j < D; j += WAVE) {
    const float g = (float)dyr[j] * gamma[j], xh = ((float)xr[j] - mu) * rs;
    float v = rs * (g - m1 - xh * m2);
    if (rr) v += (float)rr[j];
    r.dx[m * D + j] = (T)v;
  }
}

// LayerNorm backward in one pass over dy and x: dx as above (skipped when r.dx is null) and, with PARAMS, per workgroup
// the sums over its rows of dy * xhat (dgamma) and dy (dbeta).  A wavefront walks every gridDim.x * wavefronts-th row
// with the next row's loads in flight.  The wavefronts' sums are added pairwise through LDS (a fixed tree) and land in
// partial[blockIdx.x] and partial[LN_BWD_BLOCKS + blockIdx.x]; one launch adds the workgroups later.
// Bound by memory, so it needs wavefronts: 16 per workgroup (and per CU) once each of 4 would have 8 rows (25216 rows of
// 768: 64 us with 4 wavefronts per CU, 40 with 16; at 2144 rows the sums over 8 wavefronts cost 2 us more than they save).  There is one workgroup per CU whatever the row count: more workgroups
// would mean more partial rows to write, read and add.
template <typename T, int MAXC> constexpr bool many_waves() { return MAXC * Chunk<T>::V <= (sizeof(T) == 2 ? 16 : 8); }   // (by registers)
template <typename T, int MAXC, bool PARAMS>
__global__ __launch_bounds__((PARAMS && many_waves<T, MAXC>() ? 1024 : 256))
void ln_bwd_kernel(const T* __restrict__ dy, LnRows<T> r, int64_t M, int D, const float* __restrict__ mean,
                   const float* __restrict__ rstd, const float* __restrict__ gamma, float* __restrict__ partial) {
  constexpr int V = Chunk<T>::V;
  typedef typename Chunk<T>::vec vec;
  extern __shared__ float red[];            // [wavefronts / 2][2][D]
  const int lane = threadIdx.x % WAVE, w = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE), nw = blockDim.x / WAVE, nch = D / V;
  const int64_t stride = (int64_t)gridDim.x * nw;
  float gg[MAXC][V], dg[MAXC][V], db[MAXC][V];
#pragma unroll
  for (int i = 0; i < MAXC; ++i) {
    const int c = lane + i * WAVE;
#pragma unroll
    for (int e = 0; e < V; ++e) { dg[i][e] = 0.f; db[i][e] = 0.f; gg[i][e] = 0.f; }
    if (c < nch) load_params<V>(gamma + c * V, gg[i]);
  }
  vec na[MAXC], nt[MAXC];                   // the next row, already loading
  float nmu = 0.f, nrs = 0.f;
  RowPlace nplace;
  auto prefetch = [&](int64_t m) __attribute__((always_inline)) {
    if (m >= M) return;
    if (r.sc.idx && r.dx) nplace.find(r.sc, m);
#pragma unroll
    for (int i = 0; i < MAXC; ++i) {
      const int c = lane + i * WAVE;
      if (c < nch) { na[i] = *(const vec*)(dy + m * D + c * V); nt[i] = *(const vec*)(r.x + m * D + c * V); }
    }
    nmu = mean[m]; nrs = rstd[m];
  };
  int64_t m = (int64_t)blockIdx.x * nw + w;
  prefetch(m);
  for (; m < M; m += stride) {
    vec a[MAXC], t[MAXC], rr[MAXC];
#pragma unroll
    for (int i = 0; i < MAXC; ++i) { a[i] = na[i]; t[i] = nt[i]; }
    const float mu = nmu, rs = nrs;
    const RowPlace place = nplace;
    const T* res = r.dx ? res_row(r, m, D) : nullptr;
    if (res)
#pragma unroll
      for (int i = 0; i < MAXC; ++i)
        if (lane + i * WAVE < nch) rr[i] = *(const vec*)(res + (lane + i * WAVE) * V);
    prefetch(m + stride);
    float s1 = 0.f, s2 = 0.f;
#pragma unroll
    for (int i = 0; i < MAXC; ++i)
      if (lane + i * WAVE < nch)
#pragma unroll
        for (int e = 0; e < V; ++e) {
          const float d0 = (float)a[i][e], xh = ((float)t[i][e] - mu) * rs, g = d0 * gg[i][e];
          if (PARAMS) { dg[i][e] += d0 * xh; db[i][e] += d0; }
          s1 += g;
          s2 += g * xh;
        }
    if (r.dx) {
      T* out = r.sc.idx ? place.row(r, D, lane) : r.dx + m * D;
      const float m1 = wave_sum(s1) / (float)D, m2 = wave_sum(s2) / (float)D;
#pragma unroll
      for (int i = 0; i < MAXC; ++i) {
        const int c = lane + i * WAVE;
        if (c < nch) {
          vec o;
#pragma unroll
          for (int e = 0; e < V; ++e) {
            const float xh = ((float)t[i][e] - mu) * rs;
            float v = rs * ((float)a[i][e] * gg[i][e] - m1 - xh * m2);
            if (res) v += (float)rr[i][e];
            o[e] = (T)v;
          }
          *(vec*)(out + c * V) = o;
        }
      }
    }
  }
  if (!PARAMS) return;
  for (int half = nw / 2; half > 0; half /= 2) {
    if (w >= half && w < 2 * half) {
      float* p = red + (size_t)(w - half) * 2 * D;
#pragma unroll
      for (int i = 0; i < MAXC; ++i)
        if (lane + i * WAVE < nch)
#pragma unroll
          for (int e = 0; e < V; ++e) { p[(lane + i * WAVE) * V + e] = dg[i][e]; p[D + (lane + i * WAVE) * V + e] = db[i][e]; }
    }
    __syncthreads();
    if (w < half) {
      const float* p = red + (size_t)w * 2 * D;
#pragma unroll
      for (int i = 0; i < MAXC; ++i)
        if (lane + i * WAVE < nch)
#pragma unroll
          for (int e = 0; e < V; ++e) { dg[i][e] += p[(lane + i * WAVE) * V + e]; db[i][e] += p[D + (lane + i * WAVE) * V + e]; }
    }
    __syncthreads();
  }
  if (w == 0) {
    float* p0 = partial + (int64_t)blockIdx.x * D;
    float* p1 = partial + (int64_t)(LN_BWD_BLOCKS + blockIdx.x) * D;
#pragma unroll
    for (int i = 0; i < MAXC; ++i) {
      const int c = lane + i * WAVE;
      if (c < nch)
#pragma unroll
        for (int q = 0; q < V; q += 4) {
          *(float4*)(p0 + c * V + q) = make_float4(dg[i][q], dg[i][q + 1], dg[i][q + 2], dg[i][q + 3]);
          *(float4*)(p1 + c * V + q) = make_float4(db[i][q], db[i][q + 1], db[i][q + 2], db[i][q + 3]);
        }
    }
  }
}

// Pass 1 of a column reduction over M rows: block (cx, r) sums rows of chunk r for 64 columns.
// WITH_XHAT: two sums, dy*xhat (slot 0) and dy (slot 1); otherwise the plain column sum (slot 0).
template <typename T, bool WITH_XHAT>
__global__ __launch_bounds__(256) void colsum_partial_kernel(const T* __restrict__ a, int64_t ld, const T* __restrict__ x,
                                                             const float* __restrict__ mean,
                                                             const float* __restrict__ rstd, int64_t M, int N, int rows_per_chunk,
                                                             float* __restrict__ partial) {
  __shared__ float red[2][4][WAVE];
  const int lane = threadIdx.x % WAVE, w = threadIdx.x / WAVE;
  const int col = blockIdx.x * WAVE + lane;
  const int64_t r0 = (int64_t)blockIdx.y * rows_per_chunk;
  const int64_t r1 = min(r0 + (int64_t)rows_per_chunk, M);
  float s0 = 0.f, s1 = 0.f;
  if (col < N) {
    for (int64_t m = r0 + w; m < r1; m += 4) {
      const float v = (float)a[m * ld + col];
      if (WITH_XHAT) {
        s0 += v * ((float)x[m * N + col] - mean[m]) * rstd[m];
        s1 += v;
      } else {
        s0 += v;
      }
    }
  }
  red[0][w][lane] = s0;
  red[1][w][lane] = s1;
  __syncthreads();
  if (w == 0 && col < N) {
    partial[(int64_t)blockIdx.y * N + col] = red[0][0][lane] + red[0][1][lane] + red[0][2][lane] + red[0][3][lane];
    if (WITH_XHAT)
      partial[(int64_t)(COLSUM_R + blockIdx.y) * N + col] = red[1][0][lane] + red[1][1][lane] + red[1][2][lane] + red[1][3][lane];
  }
}

// Pass 2: out[col] = sum over chunks.  Wave w of the block adds chunks w, w+16, ... in ascending order, then the wave
// sums are added in wave order: a fixed order, bit-reproducible.  The second sum (if out1) starts `second` rows into
// the partial buffer.
template <bool TWO> __device__ __forceinline__ void final_columns(int col_block, const float* __restrict__ partial, int N, int chunks, int second, float* __restrict__ out0,
                                              float* __restrict__ out1) {
  __shared__ float red[2][FINAL_WAVES][WAVE];
  const int lane = threadIdx.x % WAVE, w = threadIdx.x / WAVE;
  const int col = col_block * WAVE + lane;
  float s = 0.f, t = 0.f;
  if (col < N) {
#pragma unroll 8
    for (int r = w; r < chunks; r += FINAL_WAVES) {
      s += partial[(int64_t)r * N + col];
      if (TWO) t += partial[(int64_t)(second + r) * N + col];
    }
  }
  red[0][w][lane] = s;
  red[1][w][lane] = t;
  __syncthreads();
  if (w == 0 && col < N) {
    float a0 = red[0][0][lane], a1 = red[1][0][lane];
#pragma unroll
    for (int i = 1; i < FINAL_WAVES; ++i) { a0 += red[0][i][lane]; a1 += red[1][i][lane]; }
    out0[col] = a0;
    if (TWO) out1[col] = a1;
  }
}
__global__ __launch_bounds__(FINAL_WAVES * WAVE) void colsum_final_kernel(const float* __restrict__ partial, int N, int chunks,
                                                                          int second, float* __restrict__ out0,
                                                                          float* __restrict__ out1) {
  if (out1) final_columns<true>(blockIdx.x, partial, N, chunks, second, out0, out1);
  else final_columns<false>(blockIdx.x, partial, N, chunks, second, out0, out1);
}
// What the backward pass leaves to be added up at its end, in one launch: the partials of the last weight gradient (the first `red_blocks`
// workgroups, a thread per four elements) and the same column reduction for a table of LayerNorm backward passes.
__global__ __launch_bounds__(FINAL_WAVES * WAVE) void splitk_reduce_ln_sums_kernel(int red_blocks, TnReduce red, LnDeferTable t) {
  if ((int)blockIdx.x < red_blocks) {
    const int64_t it = (int64_t)blockIdx.x * (FINAL_WAVES * WAVE) + threadIdx.x;
    if (it < splitk_reduce_items(red)) splitk_reduce_item(red, it);
    return;
  }
  const int block = blockIdx.x - red_blocks, cols = (t.D + WAVE - 1) / WAVE;
  const LnDeferEntry e = t.e[block / cols];
  final_columns<true>(block % cols, e.partial, t.D, e.blocks, LN_BWD_BLOCKS, e.dgamma, e.dbeta);
}

inline int rows_per_chunk(int64_t M) { return (int)((M + COLSUM_R - 1) / COLSUM_R); }
inline int chunks_of(int64_t M) {
  const int rpc = rows_per_chunk(M);
  return (int)((M + rpc - 1) / rpc);
}

template <typename T>
void ln_fwd(const void* x, int64_t M, int D, const float* gamma, const float* beta, float eps, void* y, float* mean, float* rstd,
            hipStream_t s) {
  const unsigned grid = (unsigned)((M + 3) / 4);
  const bool vec = with_row_chunks<T>(D, [&](auto C) {
    ln_fwd_kernel<T, decltype(C)::value><<<grid, 256, 0, s>>>((const T*)x, M, D, gamma, beta, eps, (T*)y, mean, rstd);
  });
  if (!vec) ln_fwd_any_kernel<T><<<grid, 256, 0, s>>>((const T*)x, M, D, gamma, beta, eps, (T*)y, mean, rstd);
}

// wavefronts per workgroup and workgroups of the pass with parameter sums
template <typename T, int MAXC> int bwd_waves(int64_t M) {
  return many_waves<T, MAXC>() && M >= 8 * LN_BWD_BLOCKS * 4 ? 16 : 4;
}

// false: rows this kernel does not take.  partial == null: dx only.  blocks_out: partial rows written.
template <typename T>
bool ln_bwd(const void* dy, const LnRows<T>& r, const float* mean, const float* rstd, const float* gamma, int64_t M, int D,
            float* partial, int* blocks_out, hipStream_t s) {
  return with_row_chunks<T>(D, [&](auto C) {
    constexpr int MAXC = decltype(C)::value;
    if (partial) {
      const int nw = bwd_waves<T, MAXC>(M);
      const int blocks = (int)std::min<int64_t>(LN_BWD_BLOCKS, (M + nw - 1) / nw);
      const size_t lds = sizeof(float) * nw * D;
      static bool attr_set = false;
      if (!attr_set) {
        (void)hipFuncSetAttribute((const void*)ln_bwd_kernel<T, MAXC, true>, hipFuncAttributeMaxDynamicSharedMemorySize, 64 * 1024);
        attr_set = true;
      }
      ln_bwd_kernel<T, MAXC, true><<<blocks, nw * WAVE, lds, s>>>((const T*)dy, r, M, D, mean, rstd, gamma, partial);
      *blocks_out = blocks;
    } else {
      ln_bwd_kernel<T, MAXC, false><<<(unsigned)((M + 3) / 4), 256, 0, s>>>((const T*)dy, r, M, D, mean, rstd, gamma, nullptr);
    }
  });
}

template <typename T>
void bwd_dx_t(const void* dy, const LnRows<T>& r, const float* mean, const float* rstd, const float* gamma, int64_t M, int D,
              hipStream_t s) {
  if (!r.dx) return;
  if (!ln_bwd<T>(dy, r, mean, rstd, gamma, M, D, nullptr, nullptr, s))
    ln_bwd_dx_any_kernel<T><<<(unsigned)((M + 3) / 4), 256, 0, s>>>((const T*)dy, r, M, D, mean, rstd, gamma);
}

template <typename T>
void bwd_params_t(const void* dy, const void* x, const float* mean, const float* rstd, int64_t M, int D, float* partial, float* dgamma,
                  float* dbeta, hipStream_t s) {
  const int rpc = rows_per_chunk(M), ch = chunks_of(M);
  colsum_partial_kernel<T, true><<<dim3((D + WAVE - 1) / WAVE, ch), 256, 0, s>>>((const T*)dy, D, (const T*)x, mean, rstd, M, D, rpc,
                                                                               partial);
  colsum_final_kernel<<<(D + WAVE - 1) / WAVE, FINAL_WAVES * WAVE, 0, s>>>(partial, D, ch, COLSUM_R, dgamma, dbeta);
}

template <typename T>
void bwd_t(const void* dy, const LnRows<T>& r, const float* mean, const float* rstd, const float* gamma, int64_t M, int D,
           float* partial, float* slot, float* dgamma, float* dbeta, LnDeferTable& t, hipStream_t s) {
  int blocks = 0;
  if (slot && t.count < LN_DEFER_MAX && (t.count == 0 || t.D == D) &&
      ln_bwd<T>(dy, r, mean, rstd, gamma, M, D, slot, &blocks, s)) {
    t.D = D;
    t.e[t.count++] = LnDeferEntry{slot, dgamma, dbeta, blocks};
    return;
  }
  bwd_params_t<T>(dy, r.x, mean, rstd, M, D, partial, dgamma, dbeta, s);
  bwd_dx_t<T>(dy, r, mean, rstd, gamma, M, D, s);
}

template <typename T> LnRows<T> rows_of(const void* x, const void* res, void* dx, int res_period, const LnScatter& sc) {
  return LnRows<T>{(const T*)x, (const T*)res, (T*)dx, res_period, sc};
}

}  // namespace

void layernorm_fwd(const void* x, int64_t M, int D, const float* gamma, const float* beta, float eps, bool f32, void* y, float* mean,
                   float* rstd, hipStream_t s) {
  if (M <= 0) return;
  if (f32) ln_fwd<float>(x, M, D, gamma, beta, eps, y, mean, rstd, s);
  else ln_fwd<bf16>(x, M, D, gamma, beta, eps, y, mean, rstd, s);
}

void layernorm_bwd_dx(const void* dy, const void* x, const float* mean, const float* rstd, const float* gamma, const void* res,
                      int64_t M, int D, bool f32, void* dx, hipStream_t s, int res_period, const LnScatter& sc) {
  if (M <= 0) return;
  if (f32) bwd_dx_t<float>(dy, rows_of<float>(x, res, dx, res_period, sc), mean, rstd, gamma, M, D, s);
  else bwd_dx_t<bf16>(dy, rows_of<bf16>(x, res, dx, res_period, sc), mean, rstd, gamma, M, D, s);
}

void layernorm_bwd_params(const void* dy, const void* x, const float* mean, const float* rstd, int64_t M, int D, bool f32,
                          float* partial, float* dgamma, float* dbeta, hipStream_t s) {
  if (M <= 0) return;
  if (f32) bwd_params_t<float>(dy, x, mean, rstd, M, D, partial, dgamma, dbeta, s);
  else bwd_params_t<bf16>(dy, x, mean, rstd, M, D, partial, dgamma, dbeta, s);
}

bool layernorm_bwd_scatters(int D, bool f32) { return D % (f32 ? 4 : 8) == 0 && D <= ROW_MAX; }

size_t ln_deferred_partial_floats(int D) { return (size_t)2 * LN_BWD_BLOCKS * (size_t)D; }

void layernorm_bwd(const void* dy, const void* x, const float* mean, const float* rstd, const float* gamma, const void* res, int64_t M,
                   int D, bool f32, void* dx, float* partial, float* slot, float* dgamma, float* dbeta, LnDeferTable& t, hipStream_t s,
                   int res_period, const LnScatter& sc) {
  if (M <= 0) return;
  if (f32) bwd_t<float>(dy, rows_of<float>(x, res, dx, res_period, sc), mean, rstd, gamma, M, D, partial, slot, dgamma, dbeta, t, s);
  else bwd_t<bf16>(dy, rows_of<bf16>(x, res, dx, res_period, sc), mean, rstd, gamma, M, D, partial, slot, dgamma, dbeta, t, s);
}

void ln_deferred_finish(LnDeferTable& t, const TnReduce& red, hipStream_t s) {
  constexpr int NT = FINAL_WAVES * WAVE;
  const int red_blocks = red.splits > 0 ? (int)((splitk_reduce_items(red) + NT - 1) / NT) : 0;
  const int blocks = red_blocks + t.count * ((t.D + WAVE - 1) / WAVE);
  if (blocks > 0) splitk_reduce_ln_sums_kernel<<<blocks, NT, 0, s>>>(red_blocks, red, t);
  t.count = 0;
}

size_t colsum_partial_floats(int64_t, int N) { return (size_t)2 * std::max(COLSUM_R, LN_BWD_BLOCKS) * (size_t)N; }

void colsum(const void* a, int64_t M, int N, int64_t ld, bool f32, float* partial, float* out, hipStream_t s) {
  if (M <= 0) return;
  const int rpc = rows_per_chunk(M), ch = chunks_of(M);
  const dim3 grid((N + WAVE - 1) / WAVE, ch);
  if (f32)
    colsum_partial_kernel<float, false><<<grid, 256, 0, s>>>((const float*)a, ld, nullptr, nullptr, nullptr, M, N, rpc, partial);
  else
    colsum_partial_kernel<bf16, false><<<grid, 256, 0, s>>>((const bf16*)a, ld, nullptr, nullptr, nullptr, M, N, rpc, partial);
  colsum_final_kernel<<<(N + WAVE - 1) / WAVE, FINAL_WAVES * WAVE, 0, s>>>(partial, N, ch, 0, out, nullptr);
}

}  // namespace bsr
