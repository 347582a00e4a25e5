// Element-wise kernels of the BSR step: patch extraction, the scatter that is the token gather's adjoint, losses,
// optimizer updates and weight casts.  All are HBM-bound; reductions are two-pass with a fixed order, so results are
// bit-reproducible run to run.
#include <algorithm>

#include "rowops.h"

namespace bsr {

namespace {

// ---------------------------------------------------------------- stem helpers
// out[(b*N + p), (c*P + r)*P + q] = img[b, c, gy*P + r, gx*P + q],  p = gy*G + gx
template <typename T>
__global__ void patchify_kernel(const T* __restrict__ img, int B, int C, int S, int P,
                                T* __restrict__ out) {
  const int G = S / P, Kp = C * P * P;
  const int64_t total = (int64_t)B * G * G * Kp;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
       i += (int64_t)gridDim.x * blockDim.x) {
    int kk = (int)(i % Kp);
    int64_t bp = i / Kp;
    int p = (int)(bp % (G * G));
    int b = (int)(bp / (G * G));
    int q = kk % P, r = (kk / P) % P, c = kk / (P * P);
    int gy = p / G, gx = p % G;
    out[i] = img[(((int64_t)b * C + c) * S + gy * P + r) * S + gx * P + q];
  }
}

// the same copy in 16-byte pieces: V elements of one patch row at a time (P % V == 0, 16-byte aligned rows)
// Workgroups past the copy (cls_blocks of them, one per image) write the class-token rows of the token tensor,
// x[b, 0, :] = cls + pos[0] (Sec. 3.1): the same launch, since nothing else has to run before the embedding product.
template <typename T, int V>
__global__ void patchify_vec_kernel(const T* __restrict__ img, int B, int C, int S, int P, T* __restrict__ out,
                                    int copy_blocks, const float* __restrict__ cls, const float* __restrict__ pos,
                                    int T_, int D, T* __restrict__ x) {
  if ((int)blockIdx.x >= copy_blocks) {
    const int b = blockIdx.x - copy_blocks;
    for (int j = threadIdx.x; j < D; j += blockDim.x) x[(int64_t)b * T_ * D + j] = (T)(cls[j] + pos[j]);
    return;
  }
  const int G = S / P, PV = P / V;                      // pieces per patch row
  const int64_t total = (int64_t)B * G * G * C * P * PV;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= total) return;
  const int qv = (int)(i % PV);
  int64_t t = i / PV;
  const int r = (int)(t % P); t /= P;
  const int c = (int)(t % C); t /= C;
  const int p = (int)(t % (G * G));
  const int b = (int)(t / (G * G));
  const int gy = p / G, gx = p % G;
  const uint4 v = *(const uint4*)(img + (((int64_t)b * C + c) * S + gy * P + r) * S + gx * P + qv * V);
  *(uint4*)(out + i * V) = v;                           // out index = ((b*N + p) * C*P*P + (c*P + r)*P + qv*V)
}

__global__ __launch_bounds__(256) void copy_rows_kernel(const uint4* src, uint4* dst, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) dst[i] = src[i];
}

template <typename T>
__global__ void write_cls_rows_kernel(const float* __restrict__ cls, const float* __restrict__ pos,
                                      int B, int T_, int D, T* __restrict__ x) {
  const int b = blockIdx.x;
  for (int j = threadIdx.x; j < D; j += blockDim.x) x[(int64_t)b * T_ * D + j] = (T)(cls[j] + pos[j]);
}

// Adjoint of gather + fusion: rows [CLS; kept; fused] of dy (pitch k+2) -> dx [B,T,D]; a dropped
// token j receives fw[j] times the gradient of the fused token.  Every row is written exactly once.
template <typename T>
__global__ void scatter_fused_kernel(const T* __restrict__ dy, const int32_t* __restrict__ idx,
                                     const float* __restrict__ fw, int T_, int k, int D, T* __restrict__ dx) {
  const int t = blockIdx.x, b = blockIdx.y;
  int src = -1;
  if (t == 0) {
    src = 0;
  } else {
    const int32_t* row = idx + (int64_t)b * k;
    int lo = 0, hi = k - 1;
    while (lo <= hi) {
      int mid = (lo + hi) >> 1;
      int v = row[mid];
      if (v == t - 1) { src = 1 + mid; break; }
      if (v < t - 1) lo = mid + 1; else hi = mid - 1;
    }
  }
  T* d = dx + ((int64_t)b * T_ + t) * D;
  if (src >= 0) {
    const T* s = dy + ((int64_t)b * (k + 2) + src) * D;
    for (int c = threadIdx.x; c < D; c += blockDim.x) d[c] = s[c];
  } else {
    const float wj = fw[(int64_t)b * (T_ - 1) + t - 1];
    const T* s = dy + ((int64_t)b * (k + 2) + k + 1) * D;
    for (int c = threadIdx.x; c < D; c += blockDim.x) d[c] = (T)(wj * (float)s[c]);
  }
}

// Adjoint of the gather where the LayerNorm backward does not place the rows itself (lists of the caller, rows of more than ROW_MAX): every row of
// dx is written exactly once whatever the list holds (kept rows copied, dropped rows zero), found by a binary search of the kept
// list — no atomics, no separate memset.
__global__ void scatter_rows_kernel(const uint4* __restrict__ dy, const int32_t* __restrict__ idx,
                                    int T_, int k, int row_vecs, uint4* __restrict__ dx) {
  const int t = blockIdx.x, b = blockIdx.y;
  int src = -1;
  if (t == 0) {
    src = 0;
  } else {
    const int32_t* row = idx + (int64_t)b * k;
    int lo = 0, hi = k - 1;
    while (lo <= hi) {
      int mid = (lo + hi) >> 1;
      int v = row[mid];
      if (v == t - 1) { src = 1 + mid; break; }
      if (v < t - 1) lo = mid + 1; else hi = mid - 1;
    }
  }
  uint4* d = dx + ((int64_t)b * T_ + t) * row_vecs;
  if (src < 0) {
    for (int v = threadIdx.x; v < row_vecs; v += blockDim.x) d[v] = make_uint4(0, 0, 0, 0);
  } else {
    const uint4* s = dy + ((int64_t)b * (k + 1) + src) * row_vecs;
    for (int v = threadIdx.x; v < row_vecs; v += blockDim.x) d[v] = s[v];
  }
}

// ---------------------------------------------------------------- head helpers
template <typename T>
__global__ void extract_cls_kernel(const T* __restrict__ x, int T_, int D, float* __restrict__ out) {
  const int b = blockIdx.x;
  for (int j = threadIdx.x; j < D; j += blockDim.x) out[(int64_t)b * D + j] = (float)x[(int64_t)b * T_ * D + j];
}

template <typename T>
__global__ void place_cls_grad_kernel(const float* __restrict__ dxc, int T_, int D, T* __restrict__ dx) {
  const int t = blockIdx.x, b = blockIdx.y;
  T* d = dx + ((int64_t)b * T_ + t) * D;
  for (int j = threadIdx.x; j < D; j += blockDim.x) d[j] = (t == 0) ? (T)dxc[(int64_t)b * D + j] : (T)0.f;
}

__global__ void place_rows_kernel(const uint32_t* __restrict__ rows, int words, int64_t pitch, uint32_t* __restrict__ dst) {
  for (int j = threadIdx.x; j < words; j += blockDim.x) dst[blockIdx.x * pitch + j] = rows[(int64_t)blockIdx.x * words + j];
}

// One wavefront per image: loss_b = logsumexp(z) - z[y]; dlogits = (softmax(z) - onehot) / B.
__global__ __launch_bounds__(WAVE) void cross_entropy_kernel(const float* __restrict__ logits,
                                                             const int32_t* __restrict__ labels, int B,
                                                             int C, float* __restrict__ loss_rows,
                                                             float* __restrict__ dlogits) {
  const int b = blockIdx.x, lane = threadIdx.x;
  const float* z = logits + (int64_t)b * C;
  float mx = -INFINITY;
  for (int c = lane; c < C; c += WAVE) mx = fmaxf(mx, z[c]);
  mx = wave_max(mx);
  float s = 0.f;
  for (int c = lane; c < C; c += WAVE) s += expf(z[c] - mx);
  const float lse = mx + logf(wave_sum(s));
  const int y = labels[b];
  if (lane == 0) loss_rows[b] = lse - ((y >= 0 && y < C) ? z[y] : 0.f);
  for (int c = lane; c < C; c += WAVE)
    dlogits[(int64_t)b * C + c] = (expf(z[c] - lse) - (c == y ? 1.f : 0.f)) / (float)B;
}

// one wavefront: lane l adds v[l], v[l + 64], ..., then the lanes are added as a tree (10 us for 256 values by one thread)
__global__ __launch_bounds__(WAVE) void mean_of_rows_kernel(const float* __restrict__ v, int n, float scale, float* __restrict__ out) {
  float s = 0.f;
  for (int i = threadIdx.x; i < n; i += WAVE) s += v[i];
  s = wave_sum(s);
  if (threadIdx.x == 0) *out = s * scale;
}

constexpr int MSQ_BLOCKS = 256;
template <typename T>
__global__ __launch_bounds__(256) void mean_sq_kernel(const T* __restrict__ x, int64_t n,
                                                      float* __restrict__ partial, T* __restrict__ dx) {
  __shared__ float red[4];
  const int64_t per = (n + MSQ_BLOCKS - 1) / MSQ_BLOCKS;
  const int64_t i0 = (int64_t)blockIdx.x * per, i1 = min(i0 + per, n);
  const float g = 2.0f / (float)n;
  float s = 0.f;
  for (int64_t i = i0 + threadIdx.x; i < i1; i += blockDim.x) {
    float v = (float)x[i];
    s += v * v;
    if (dx) dx[i] = (T)(v * g);
  }
  s = wave_sum(s);
  if (threadIdx.x % WAVE == 0) red[threadIdx.x / WAVE] = s;
  __syncthreads();
  if (threadIdx.x == 0) partial[blockIdx.x] = red[0] + red[1] + red[2] + red[3];
}

// ---------------------------------------------------------------- weights: casts and SGD
// A table of matrices (and small tensors) in one launch.  64x64 tiles, 16-byte accesses; the tile goes through LDS so
// that both the straight [rows,cols] and the transposed [cols,rows] bf16 copies are written with
// contiguous rows.  With UPDATE the tile is first updated by SGD (Sec. 5 of the paper):
//   g' = g + wd*w;  mu > 0: m = mu*m + g', w -= lr*m;  else w -= lr*g'.
// rows and cols are multiples of 4.
typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));

// one element of the optimiser update; m / v2 are the element's moments, used and rewritten only by
// the rules that have them
__device__ inline float opt_update(const OptArgs& o, float w, float g, float& m, float& v2) {
  if (o.kind == OPT_ADAMW) {
    m = o.b1 * m + (1.0f - o.b1) * g;
    v2 = o.b2 * v2 + (1.0f - o.b2) * g * g;
    return w - o.lr * ((m / o.bc1) / (sqrtf(v2 / o.bc2) + o.eps) + o.wd * w);
  }
  float gp = g + o.wd * w;
  if (o.mu > 0.f) {
    gp = o.mu * m + gp;
    m = gp;
  }
  return w - o.lr * gp;
}

// four consecutive elements at offset off (16-byte accesses)
__device__ inline float4 opt_update4(const OptArgs& o, float4 w, float4 g, float* m, float* v2, int64_t off) {
  const bool use_m = o.kind == OPT_ADAMW || o.mu > 0.f, use_v = o.kind == OPT_ADAMW;
  float4 mm = use_m ? *(const float4*)(m + off) : make_float4(0.f, 0.f, 0.f, 0.f);
  float4 vv = use_v ? *(const float4*)(v2 + off) : make_float4(0.f, 0.f, 0.f, 0.f);
  w.x = opt_update(o, w.x, g.x, mm.x, vv.x);
  w.y = opt_update(o, w.y, g.y, mm.y, vv.y);
  w.z = opt_update(o, w.z, g.z, mm.z, vv.z);
  w.w = opt_update(o, w.w, g.w, mm.w, vv.w);
  if (use_m) *(float4*)(m + off) = mm;
  if (use_v) *(float4*)(v2 + off) = vv;
  return w;
}

constexpr int VEC_PER_BLOCK = 1024;
// the entry whose workgroups hold block: a lane per entry (walking the table one scalar load after the other, a workgroup began up to 16
// of them late)
__device__ inline int table_entry(const int* start, int count, int block) {
  const int lane = threadIdx.x % WAVE;
  return __builtin_amdgcn_readfirstlane(__popcll(__ballot(lane < count && block >= start[min(lane, count - 1)])) - 1);
}
static_assert(OPT_MATS <= WAVE && OPT_VECS <= WAVE, "a lane per entry");

template <bool UPDATE>
__global__ __launch_bounds__(256) void opt_table_kernel(OptTable t, OptArgs o) {
  __shared__ float tile[64][65];
  if (UPDATE && (int)blockIdx.x >= t.mat_blocks) {       // a slice of a small tensor
    const int block = blockIdx.x - t.mat_blocks, ei = table_entry(t.vec_start, t.vecs, block);
    const VecEntry e = t.vec[ei];
    const int64_t i0 = (int64_t)(block - t.vec_start[ei]) * VEC_PER_BLOCK + threadIdx.x;
#pragma unroll
    for (int j = 0; j < VEC_PER_BLOCK / 256; ++j) {
      const int64_t i = i0 + 256 * j;
      if (i >= e.n) break;
      const bool use_m = o.kind == OPT_ADAMW || o.mu > 0.f, use_v = o.kind == OPT_ADAMW;
      float mm = use_m ? e.m[i] : 0.f, vv = use_v ? e.v2[i] : 0.f;
      e.w[i] = opt_update(o, e.w[i], e.g[i], mm, vv);
      if (use_m) e.m[i] = mm;
      if (use_v) e.v2[i] = vv;
    }
    return;
  }
  const int ei = table_entry(t.mat_start, t.mats, blockIdx.x);
  MatEntry e = t.mat[ei];
  const int tiles_x = (e.cols + 63) / 64, tiles = tiles_x * ((e.rows + 63) / 64), which = (blockIdx.x - t.mat_start[ei]) / tiles;
  const int local = blockIdx.x - t.mat_start[ei] - which * tiles;
  if (which > 0) {                                        // (uniform)
    const int64_t at = (int64_t)which * e.rows * e.cols;
    e.w += at;
    if (e.g) e.g += at;
    if (e.m) e.m += at;
    if (e.v2) e.v2 += at;
    if (e.s) e.s += at;
    if (e.t) e.t += at;
  }
  const int c0 = (local % tiles_x) * 64, r0 = (local / tiles_x) * 64;
  const int tx = threadIdx.x % 16, ty = threadIdx.x / 16;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int lr_ = ty + 16 * i, r = r0 + lr_, c = c0 + 4 * tx;
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    if (r < e.rows && c < e.cols) {
      const int64_t off = (int64_t)r * e.cols + c;
      v = *(const float4*)(e.w + off);
      if (UPDATE) {
        const float4 g = *(const float4*)(e.g + off);
        v = opt_update4(o, v, g, e.m, e.v2, off);
        *(float4*)(e.w + off) = v;
      }
      if (e.s) {
        bf16x4_t o;
        o[0] = (bf16)v.x; o[1] = (bf16)v.y; o[2] = (bf16)v.z; o[3] = (bf16)v.w;
        *(bf16x4_t*)(e.s + off) = o;
      }
    }
    tile[lr_][4 * tx + 0] = v.x; tile[lr_][4 * tx + 1] = v.y; tile[lr_][4 * tx + 2] = v.z; tile[lr_][4 * tx + 3] = v.w;
  }
  __syncthreads();
  if (e.t) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int cc = ty + 16 * i, c = c0 + cc, r = r0 + 4 * tx;
      if (c < e.cols && r < e.rows) {
        bf16x4_t o;
#pragma unroll
        for (int j = 0; j < 4; ++j) o[j] = (bf16)tile[4 * tx + j][cc];
        *(bf16x4_t*)(e.t + (int64_t)c * e.rows + r) = o;
      }
    }
  }
}

// LayerNorm folded into the frozen linear layer behind it: one thread per output column n walks k in
// ascending order, so the column sum is the sum of exactly the rounded values the matrix cores will see.
__global__ __launch_bounds__(128) void ln_fold_kernel(const float* __restrict__ w, const float* __restrict__ bias,
                                                     const float* __restrict__ gamma, const float* __restrict__ beta,
                                                     int in, int out, bf16* __restrict__ w_t, float* __restrict__ colsum,
                                                     float* __restrict__ bias_out) {
  const int n = blockIdx.x * blockDim.x + threadIdx.x;
  if (n >= out) return;
  float cs = 0.f, bb = bias[n];
  for (int k0 = 0; k0 < in; k0 += 8) {
    Chunk<bf16>::vec o;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const float wv = w[(int64_t)(k0 + j) * out + n];
      const bf16 r = (bf16)(wv * gamma[k0 + j]);
      o[j] = r;
      cs += (float)r;
      bb = fmaf(beta[k0 + j], wv, bb);
    }
    *(Chunk<bf16>::vec*)(w_t + (int64_t)n * in + k0) = o;
  }
  colsum[n] = cs;
  bias_out[n] = bb;
}

}  // namespace

// ---------------------------------------------------------------- launchers

void patchify(const void* img, int B, int C, int S, int P, bool f32, void* out, hipStream_t s, const float* cls,
              const float* pos, int T, int D, void* x) {
  const int64_t total = (int64_t)B * C * S * S;
  const int V = f32 ? 4 : 8;                             // elements per 16 bytes
  if (P % V == 0 && S % V == 0 && (((uintptr_t)img | (uintptr_t)out) & 15) == 0) {
    const unsigned vgrid = (unsigned)((total / V + 255) / 256), extra = cls ? (unsigned)B : 0u;
    if (f32) patchify_vec_kernel<float, 4><<<vgrid + extra, 256, 0, s>>>((const float*)img, B, C, S, P, (float*)out, (int)vgrid, cls, pos, T, D, (float*)x);
    else patchify_vec_kernel<bf16, 8><<<vgrid + extra, 256, 0, s>>>((const bf16*)img, B, C, S, P, (bf16*)out, (int)vgrid, cls, pos, T, D, (bf16*)x);
    return;
  }
  const unsigned grid = (unsigned)std::min<int64_t>((total + 255) / 256, 65536);
  if (f32) patchify_kernel<float><<<grid, 256, 0, s>>>((const float*)img, B, C, S, P, (float*)out);
  else patchify_kernel<bf16><<<grid, 256, 0, s>>>((const bf16*)img, B, C, S, P, (bf16*)out);
  if (cls) write_cls_rows(cls, pos, B, T, D, f32, x, s);
}

void copy_rows(const void* src, void* dst, size_t bytes, hipStream_t s) {
  const int64_t n = (int64_t)(bytes / 16);
  if (n > 0) copy_rows_kernel<<<(unsigned)((n + 255) / 256), 256, 0, s>>>((const uint4*)src, (uint4*)dst, n);
}

void write_cls_rows(const float* cls, const float* pos, int B, int T, int D, bool f32, void* x,
                    hipStream_t s) {
  if (f32) write_cls_rows_kernel<float><<<B, 256, 0, s>>>(cls, pos, B, T, D, (float*)x);
  else write_cls_rows_kernel<bf16><<<B, 256, 0, s>>>(cls, pos, B, T, D, (bf16*)x);
}

void scatter_tokens(const void* dy, const int32_t* idx, int B, int T, int k, int D, bool f32,
                    void* dx, hipStream_t s, const float* fw) {
  if (fw) {   // rows of dy are [CLS; kept; fused]
    if (f32) scatter_fused_kernel<float><<<dim3(T, B), 128, 0, s>>>((const float*)dy, idx, fw, T, k, D, (float*)dx);
    else scatter_fused_kernel<bf16><<<dim3(T, B), 128, 0, s>>>((const bf16*)dy, idx, fw, T, k, D, (bf16*)dx);
    return;
  }
  const int row_vecs = D * (f32 ? 4 : 2) / 16;
  scatter_rows_kernel<<<dim3(T, B), 64, 0, s>>>((const uint4*)dy, idx, T, k, row_vecs, (uint4*)dx);
}

void extract_cls(const void* x, int B, int T, int D, bool f32, float* out, hipStream_t s) {
  if (f32) extract_cls_kernel<float><<<B, 256, 0, s>>>((const float*)x, T, D, out);
  else extract_cls_kernel<bf16><<<B, 256, 0, s>>>((const bf16*)x, T, D, out);
}

void place_cls_grad(const float* dxc, int B, int T, int D, bool f32, void* dx, hipStream_t s) {
  if (f32) place_cls_grad_kernel<float><<<dim3(T, B), 128, 0, s>>>(dxc, T, D, (float*)dx);
  else place_cls_grad_kernel<bf16><<<dim3(T, B), 128, 0, s>>>(dxc, T, D, (bf16*)dx);
}

void place_rows(const void* rows, int n, size_t row_bytes, int64_t every, void* dst, hipStream_t s) {
  const int words = (int)(row_bytes / 4);
  place_rows_kernel<<<n, words < 256 ? 64 : 256, 0, s>>>((const uint32_t*)rows, words, every * words, (uint32_t*)dst);
}

void cross_entropy(const float* logits, const int32_t* labels, int B, int C, float* loss_rows,
                   float* dlogits, float* loss, hipStream_t s) {
  cross_entropy_kernel<<<B, WAVE, 0, s>>>(logits, labels, B, C, loss_rows, dlogits);
  mean_of_rows_kernel<<<1, 64, 0, s>>>(loss_rows, B, 1.0f / (float)B, loss);
}

size_t mean_sq_partial_floats() { return MSQ_BLOCKS; }

void mean_sq_loss(const void* x, int64_t n, bool f32, float* partial, float* loss, void* dx,
                  hipStream_t s) {
  if (f32) mean_sq_kernel<float><<<MSQ_BLOCKS, 256, 0, s>>>((const float*)x, n, partial, (float*)dx);
  else mean_sq_kernel<bf16><<<MSQ_BLOCKS, 256, 0, s>>>((const bf16*)x, n, partial, (bf16*)dx);
  mean_of_rows_kernel<<<1, 64, 0, s>>>(partial, MSQ_BLOCKS, 1.0f / (float)n, loss);
}

void ln_fold_weights(const float* w, const float* bias, const float* gamma, const float* beta, int in, int out,
                     bf16* w_t, float* colsum, float* bias_out, hipStream_t s) {
  ln_fold_kernel<<<(out + 127) / 128, 128, 0, s>>>(w, bias, gamma, beta, in, out, w_t, colsum, bias_out);
}

void opt_run(OptTable& t, bool update, const OptArgs& o, hipStream_t s) {
  const int blocks = t.mat_blocks + t.vec_blocks;
  if (blocks > 0) {
    if (update) opt_table_kernel<true><<<blocks, 256, 0, s>>>(t, o);
    else opt_table_kernel<false><<<blocks, 256, 0, s>>>(t, OptArgs());
  }
  t.mats = t.vecs = t.mat_blocks = t.vec_blocks = 0;
}

void opt_add_mat(OptTable& t, const MatEntry& e, bool update, const OptArgs& o, hipStream_t s) {
  if (t.mats == OPT_MATS) opt_run(t, update, o, s);
  t.mat[t.mats] = e;
  t.mat_start[t.mats++] = t.mat_blocks;
  t.mat_blocks += e.count * ((e.rows + 63) / 64) * ((e.cols + 63) / 64);
}

void opt_add_vec(OptTable& t, const VecEntry& e, bool update, const OptArgs& o, hipStream_t s) {
  if (t.vecs == OPT_VECS) opt_run(t, update, o, s);
  t.vec[t.vecs] = e;
  t.vec_start[t.vecs++] = t.vec_blocks;
  t.vec_blocks += (int)((e.n + VEC_PER_BLOCK - 1) / VEC_PER_BLOCK);
}

}  // namespace bsr
