// Classification head of the fine-tuning step in two launches (Sec. 3.1: the class token feeds the
// classifier; the loss is the batch mean of the cross-entropy):
//   head_rows_kernel   one workgroup per image: final LayerNorm of the class token, logits, loss of the
//                      image, dlogits = (softmax - onehot) / B, dz = dlogits . W_h^T, the LayerNorm
//                      backward of that row, and the gradient at the last block's output (the class
//                      row gets it; further workgroups set the other token rows to zero);
//   head_batch_kernel  the sums over the batch: loss, dW_h = z^T dlogits, db_h, dgamma_f, dbeta_f,
//                      each in a fixed order (bit-reproducible).
// All arithmetic is fp32 whatever the activation type.
// Bound by latency: an image's workgroup reads W_h once (307 KB at 768 x 100, from L2) or, beyond what its registers hold, twice.
// Both passes walk W_h as it lies in memory, VEC classes per load, as many rows at once as the 1024 threads cover; what is to be
// added across threads goes through LDS.  A thread's first rows (20 of four classes: all of 768 x 100; 40 of one: 384 x 102 takes 39, 768 x 101 77)
// are asked for in one go ahead of the LayerNorm and kept for dz, the others eight (of four classes five) at a time with the last batch filled up by
// repeats, where loops of eight left up to seven rows to be waited for one by one, in every chunk of dz again.  A thread's 48 rows of one class held: as long within
// 1 %, 10 classes 1.02 times; 14 of the others asked for together 1.02 .. 1.05.  Head launches in a graph, loops of eight -> this, 32 images: 768 x 100 21.1 -> 18.6 us,
// 768 x 102 39.7 -> 31.4, 768 x 37 20.6 -> 18.8, 768 x 10 16.1 -> 14.4, 384 x 102 25.7 -> 20.5, 384 x 100 16.7 -> 15.5, 384 x 10 13.6 -> 13.4, 1024 x 101 40.0 -> 38.3.
// dz takes eight rows a thread between two barriers, as those loops did: with the five or seven asked for together between two barriers, and four
// values for every sum of at most eight, 192 x 120 had become 1.03, 768 x 28 1.06, 1024 x 20 1.06, 384 x 56 1.03 and 1024 x 101 1.02 times as long as those loops.
// (Lanes along the classes with a wave sum per row of W_h: 32 us at 32 images, 768 x 100.
// The batch kernel with a thread per element walking all images: 13 us at 32 images, 48 at 128; now 6 and 17.)
#include "rowops.h"

#include <stdint.h>

#include <type_traits>

namespace bsr {
namespace {

constexpr int HT = 1024, HW = HT / WAVE;               // threads and wavefronts per workgroup of the row kernel
constexpr int SCRATCH = 9216, TAKES_SCRATCH = 8192;    // floats of LDS for partial sums; those that decide which heads come here
// (Registers: 118 of 128 at 20 rows of four classes, 21 in chunks of seven spill; 65 at 40 of one.)
constexpr int CHUNK4 = 5, CHUNK1 = 8;                  // rows of W_h (of four classes, of one) that a thread of the row kernel asks for together
constexpr int HELD4 = 4 * CHUNK4, HELD1 = 5 * CHUNK1;  // and those it holds in registers from the logits to dz
constexpr int SUM = 8;                                 // held rows between two barriers of dz
static_assert(SUM * 1152 <= SCRATCH && CHUNK4 <= SUM && CHUNK1 <= SUM, "R rows at the pitch of dz are at most 128 x 9 numbers");
constexpr int WIDE_G = 128, PARTS = 8;                 // groups of VEC classes that make a wide head; its ranges of rows
constexpr int ZERO_PARTS = 4;                          // workgroups per image that clear the other token rows
constexpr int BT = 256;                                // threads per workgroup of the batch kernel
constexpr int TD = 16, TC = 64, BCH = 32;              // batch kernel: rows x classes of W_h per workgroup, images per chunk

// sum (or max) over the workgroup; every thread gets the result; red: HW floats of LDS
__device__ inline float block_sum(float v, float* red) {
  v = wave_sum(v);
  __syncthreads();
  if (threadIdx.x % WAVE == 0) red[threadIdx.x / WAVE] = v;
  __syncthreads();
  float s = red[0];
#pragma unroll
  for (int i = 1; i < HW; ++i) s += red[i];
  return s;
}
__device__ inline float block_max(float v, float* red) {
  v = wave_max(v);
  __syncthreads();
  if (threadIdx.x % WAVE == 0) red[threadIdx.x / WAVE] = v;
  __syncthreads();
  float s = red[0];
#pragma unroll
  for (int i = 1; i < HW; ++i) s = fmaxf(s, red[i]);
  return s;
}

template <typename T>
__device__ __forceinline__ void zero_rows(T* dst, int64_t n, int part) {
  if ((((uintptr_t)dst) & 15) == 0 && (n * sizeof(T)) % 16 == 0) {
    uint4* z = (uint4*)dst;
    const int64_t nv = n * sizeof(T) / 16;
    for (int64_t i = (int64_t)part * HT + threadIdx.x; i < nv; i += ZERO_PARTS * HT) z[i] = make_uint4(0u, 0u, 0u, 0u);
  } else {
    for (int64_t i = (int64_t)part * HT + threadIdx.x; i < n; i += ZERO_PARTS * HT) dst[i] = (T)0.f;
  }
}

// v[tid % 8], v[tid % 8 + 8], ... of n values `step` apart, added in that order; behind the first, four at a time are read together
__device__ __forceinline__ float every_eighth(const float* v, int step, int n) {
  const int first = threadIdx.x & 7;
  float a = first < n ? 0.f + v[first * step] : 0.f;
  for (int i = first + 8; i < n; i += 32) {
    float t[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) t[j] = v[min(i + 8 * j, n - 1) * step];
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (i + 8 * j < n) a += t[j];
  }
  return a;
}

// a value the compiler works out addresses from again, where it would keep those of every row in registers
__device__ __forceinline__ int anew(int v) {
  asm volatile("" : "+v"(v));
  return v;
}

template <typename T, int VEC, bool WIDE>
__global__ __launch_bounds__(HT) void head_rows_kernel(const T* __restrict__ x, int Tl, int D, int C, int B,
                                                       const float* __restrict__ gamma, const float* __restrict__ beta,
                                                       float eps, const float* __restrict__ w_head,
                                                       const float* __restrict__ b_head, const int32_t* __restrict__ labels,
                                                       float* __restrict__ xhat_out, float* __restrict__ z_out,
                                                       float* __restrict__ logits_out, float* __restrict__ dlogits_out,
                                                       float* __restrict__ dz_out, float* __restrict__ loss_rows,
                                                       T* __restrict__ dx) {
  extern __shared__ float sm[];
  const int b = blockIdx.x, tid = threadIdx.x;
  if (blockIdx.y > 0) {           // the other token rows of this image receive no gradient from the head
    zero_rows(dx + ((int64_t)b * Tl + 1) * D, (int64_t)(Tl - 1) * D, blockIdx.y - 1);
    return;
  }
  typedef float vecf __attribute__((ext_vector_type(VEC)));
  float* xh = sm;                 // [D] normalised class token
  float* zs = xh + D;             // [D] LayerNorm output, later dz
  float* lg = zs + D;             // [C] logits, then dlogits
  float* red = lg + C;            // [HW]
  float* scr = red + HW;          // [SCRATCH] partial sums
  const T* xr = x + (int64_t)b * Tl * D;
  // G groups of VEC classes, R rows of W_h at a time: thread (r, group) takes rows r, r + R, ... both for the logits and for dz.
  // Its first HELD rows are asked for ahead of the LayerNorm and stay for dz; a row past the last reads the last and counts nowhere.
  constexpr int HELD = VEC == 4 ? HELD4 : HELD1, CHUNK = VEC == 4 ? CHUNK4 : CHUNK1;
  const int G = C / VEC, R = WIDE ? PARTS : max(1, HT / G), first = tid / G, grp = tid % G;
  vecf held[WIDE ? 1 : HELD];
  auto rows_of = [&](vecf* w, int k0) {
    const int row = anew(first);
#pragma unroll
    for (int j = 0; j < CHUNK; ++j) w[j] = *(const vecf*)(w_head + (uint32_t)(min(row + (k0 + j) * R, D - 1) * C + grp * VEC));
  };
  // final LayerNorm of the class token (two passes over the row held in LDS)
  float s = 0.f;
  for (int d = tid; d < D; d += HT) { const float v = (float)xr[d]; xh[d] = v; s += v; }
  const int early_y = WIDE ? 0 : labels[b];      // (WIDE: no other loads ahead that its wait could hide behind)
  if constexpr (!WIDE) {
#pragma unroll
    for (int k = 0; k < HELD; k += CHUNK) {
      if (k * R < D) rows_of(held + k, k);
      else
#pragma unroll
        for (int j = 0; j < CHUNK; ++j) held[k + j] = (vecf)0.f;
    }
  }
  const float mean = block_sum(s, red) / (float)D;
  float q = 0.f;
  for (int d = tid; d < D; d += HT) { const float v = xh[d] - mean; q += v * v; }
  const float rstd = rsqrtf(block_sum(q, red) / (float)D + eps);
  for (int d = tid; d < D; d += HT) {
    const float h = (xh[d] - mean) * rstd, z = h * gamma[d] + beta[d];
    xh[d] = h; zs[d] = z;
    xhat_out[(int64_t)b * D + d] = h;
    z_out[(int64_t)b * D + d] = z;
  }
  __syncthreads();
  // logits: thread (r, group) adds up its rows.  WIDE: a wavefront adds up one of R ranges of rows, its lanes along the classes,
  // 64 groups at a time.
  if constexpr (WIDE) {
    const int part = tid / WAVE % PARTS, n = D / PARTS;           // (D is a multiple of 8)
    for (int g = tid / WAVE / PARTS * WAVE + tid % WAVE; g < G; g += HT / PARTS) {
      const float* wp = w_head + (int64_t)part * n * C + g * VEC;
      vecf a = (vecf)0.f;
#pragma unroll 8
      for (int d = 0; d < n; ++d) a += zs[part * n + d] * *(const vecf*)(wp + (int64_t)d * C);
#pragma unroll
      for (int v = 0; v < VEC; ++v) scr[part * C + g * VEC + v] = a[v];
    }
  } else {
    vecf a = (vecf)0.f;
    auto add = [&](const vecf* w, int k0) {
      const int row = anew(first);
#pragma unroll
      for (int j = 0; j < CHUNK; ++j) {
        const int d = row + (k0 + j) * R;
        if (d < D) a += zs[d] * w[j];
      }
    };
#pragma unroll
    for (int k = 0; k < HELD; k += CHUNK)
      if (k * R < D) add(held + k, k);
    for (int k = HELD; k * R < D; k += CHUNK) {
      vecf w[CHUNK];
      rows_of(w, k);
      add(w, k);
    }
    if (first < R)
#pragma unroll
      for (int v = 0; v < VEC; ++v) scr[first * C + grp * VEC + v] = a[v];
  }
  __syncthreads();
  for (int i = tid / 8; i < C; i += HT / 8) {          // eight threads per class
    float a = eight_sum(every_eighth(scr + i, C, R));
    if ((tid & 7) == 0) {
      if (b_head) a += b_head[i];
      lg[i] = a;
      logits_out[(int64_t)b * C + i] = a;
    }
  }
  __syncthreads();
  // cross-entropy of this image and dlogits
  float mx = -INFINITY;
  for (int c = tid; c < C; c += HT) mx = fmaxf(mx, lg[c]);
  mx = block_max(mx, red);
  float se = 0.f;
  for (int c = tid; c < C; c += HT) se += expf(lg[c] - mx);
  const float lse = mx + logf(block_sum(se, red));
  const int y = WIDE ? labels[b] : early_y;
  if (tid == 0) loss_rows[b] = lse - ((y >= 0 && y < C) ? lg[y] : 0.f);
  __syncthreads();
  for (int c = tid; c < C; c += HT) {
    const float g = (expf(lg[c] - lse) - (c == y ? 1.f : 0.f)) / (float)B;
    lg[c] = g;
    dlogits_out[(int64_t)b * C + c] = g;
  }
  __syncthreads();
  // dz = dlogits . W_h^T: the same walk, SUM R rows at a time of those held, CHUNK R of the others; each thread leaves the product of its
  // VEC classes, then eight threads add up a row (odd pitch from eight groups on).
  // WIDE (a chunk would be a few rows, and adding them up all there is): a wavefront takes four rows at a time, its lanes along
  // the classes.
  if constexpr (WIDE) {
    for (int d0 = tid / WAVE * 4; d0 < D; d0 += HW * 4) {
      float a[4] = {0.f, 0.f, 0.f, 0.f};
      const float* wp = w_head + (int64_t)d0 * C;
#pragma unroll 4
      for (int g = tid % WAVE; g < G; g += WAVE) {
        const vecf dl = *(const vecf*)(lg + g * VEC);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const vecf w = *(const vecf*)(wp + (int64_t)i * C + g * VEC);
#pragma unroll
          for (int v = 0; v < VEC; ++v) a[i] = fmaf(dl[v], w[v], a[i]);
        }
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        a[i] = wave_sum(a[i]);
        if (tid % WAVE == 0) zs[d0 + i] = a[i];          // raw dz (z is not needed any more)
      }
    }
    __syncthreads();
  } else {
    const int GP = G < 8 ? G : G | 1;
    float dl[VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) dl[v] = lg[grp * VEC + v];
    auto chunk = [&](const vecf* w, int k0, auto n) {
      constexpr int N = decltype(n)::value;
      const int d0 = k0 * R, rows = min(N * R, D - d0), row = anew(first);
#pragma unroll
      for (int j = 0; j < N; ++j) {
        const int r = row + j * R;
        float a = 0.f;
#pragma unroll
        for (int v = 0; v < VEC; ++v) a = fmaf(dl[v], w[j][v], a);
        if (row < R && r < rows) scr[r * GP + grp] = a;
      }
      __syncthreads();
      for (int r = tid / 8; r < rows; r += HT / 8) {
        const float a = eight_sum(every_eighth(scr + r * GP, 1, G));
        if ((tid & 7) == 0) zs[d0 + r] = a;
      }
      __syncthreads();
    };
    constexpr std::integral_constant<int, SUM> some{};
#pragma unroll
    for (int k = 0; k + SUM <= HELD; k += SUM)
      if (k * R < D) chunk(held + k, k, some);
    if constexpr (HELD % SUM)
      if (HELD / SUM * SUM * R < D) chunk(held + HELD / SUM * SUM, HELD / SUM * SUM, std::integral_constant<int, HELD % SUM>{});
    for (int k = HELD; k * R < D; k += CHUNK) {
      vecf w[CHUNK];
      rows_of(w, k);
      chunk(w, k, std::integral_constant<int, CHUNK>{});
    }
  }
  // the LayerNorm backward of the row:
  //   dxhat = dz * gamma;  dx = rstd * (dxhat - mean(dxhat) - xhat * mean(dxhat * xhat))
  float s1 = 0.f, s2 = 0.f;
  for (int d = tid; d < D; d += HT) {
    const float t = zs[d];
    dz_out[(int64_t)b * D + d] = t;
    const float dh = t * gamma[d];                       // dxhat
    zs[d] = dh;
    s1 += dh;
    s2 += dh * xh[d];
  }
  s1 = block_sum(s1, red) / (float)D;
  s2 = block_sum(s2, red) / (float)D;
  T* dr = dx + (int64_t)b * Tl * D;
  for (int d = tid; d < D; d += HT) dr[d] = (T)(rstd * (zs[d] - s1 - xh[d] * s2));
}

// Workgroups [0, nw): a TD x TC piece of dW_h, the images through LDS BCH at a time, added in ascending order;
// [nw, nw + D / 64): dgamma_f, dbeta_f of 64 features (four threads each take every fourth image); the last: db_h, loss.
__global__ __launch_bounds__(BT) void head_batch_kernel(const float* __restrict__ z, const float* __restrict__ xhat,
                                                        const float* __restrict__ dlogits, const float* __restrict__ dz,
                                                        const float* __restrict__ loss_rows, int B, int D, int C, int nw,
                                                        float* __restrict__ dw, float* __restrict__ db,
                                                        float* __restrict__ dgamma, float* __restrict__ dbeta,
                                                        float* __restrict__ loss) {
  __shared__ __attribute__((aligned(16))) float zs[BCH][TD];
  __shared__ float ls[BCH][TC];
  const int tid = threadIdx.x, lane = tid % WAVE, w = tid / WAVE;
  if ((int)blockIdx.x < nw) {
    const int ntc = (C + TC - 1) / TC, d0 = (blockIdx.x / ntc) * TD, c0 = (blockIdx.x % ntc) * TC;
    float a[4] = {0.f, 0.f, 0.f, 0.f};                 // rows d0 + 4 w .. + 3, class c0 + lane
    for (int b0 = 0; b0 < B; b0 += BCH) {
      if (b0) __syncthreads();
      const int nb = min(BCH, B - b0);
      for (int i = tid; i < nb * TD; i += BT) { const int d = d0 + i % TD; zs[i / TD][i % TD] = d < D ? z[(int64_t)(b0 + i / TD) * D + d] : 0.f; }
      for (int i = tid; i < nb * TC; i += BT) { const int c = c0 + i % TC; ls[i / TC][i % TC] = c < C ? dlogits[(int64_t)(b0 + i / TC) * C + c] : 0.f; }
      __syncthreads();
#pragma unroll 4
      for (int b = 0; b < nb; ++b) {
        const float g = ls[b][lane];
        const float4 v = *(const float4*)&zs[b][4 * w];
        a[0] = fmaf(v.x, g, a[0]); a[1] = fmaf(v.y, g, a[1]); a[2] = fmaf(v.z, g, a[2]); a[3] = fmaf(v.w, g, a[3]);
      }
    }
    if (c0 + lane < C)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (d0 + 4 * w + i < D) dw[(int64_t)(d0 + 4 * w + i) * C + c0 + lane] = a[i];
    return;
  }
  const int d0 = (blockIdx.x - nw) * WAVE;
  float* r0 = &ls[0][0];
  if (d0 < D) {
    const int d = d0 + lane;
    float g = 0.f, bt = 0.f;
    if (d < D)
#pragma unroll 8
      for (int b = w; b < B; b += BT / WAVE) {
        const float v = dz[(int64_t)b * D + d];
        g = fmaf(v, xhat[(int64_t)b * D + d], g);
        bt += v;
      }
    r0[tid] = g;
    r0[BT + tid] = bt;
    __syncthreads();
    if (w == 0 && d < D) {
#pragma unroll
      for (int i = 1; i < BT / WAVE; ++i) { g += r0[i * WAVE + lane]; bt += r0[BT + i * WAVE + lane]; }
      dgamma[d] = g;
      dbeta[d] = bt;
    }
    return;
  }
  if (db)
    for (int c = tid; c < C; c += BT) {
      float a = 0.f;
#pragma unroll 16
      for (int b = 0; b < B; ++b) a += dlogits[(int64_t)b * C + c];
      db[c] = a;
    }
  if (w == 0) {
    float a = 0.f;
    for (int b = lane; b < B; b += WAVE) a += loss_rows[b];
    a = wave_sum(a);
    if (lane == 0) *loss = a / (float)B;
  }
}

}  // namespace

static bool four_classes(int C, const float* w_head) { return C % 4 == 0 && ((uintptr_t)w_head & 15) == 0; }   // (as rows of W_h start)
static bool wide_head(int C, const float* w_head) { return C / (four_classes(C, w_head) ? 4 : 1) >= WIDE_G; }
static size_t head_lds_bytes(int D, int C, const float* w_head, int scratch) {
  return sizeof(float) * ((size_t)2 * D + (size_t)C + HW + (wide_head(C, w_head) ? (size_t)PARTS * C : (size_t)scratch));
}

// Whether these kernels take a head, or the general ones do (products of their own, which share W_h among all CUs where here
// every image's workgroup reads all of it): by LDS, then by what is faster.  Steps of a small model, here / general, in us:
// 768 x 300 113 .. 169 / 120 .. 162 at 1 .. 128 images, 768 x 600 149 .. 203 / 126 .. 167, 384 x 1000 112 .. 164 /
// 114 .. 147, 192 x 1640 101 .. 151 / 120 .. 152.  Where the classes are no multiple of four the general products go without
// the matrix cores and take longer by the image: 768 x 1301 256 .. 317 / 132 .. 602, equal at 40.
bool head_takes(int B, int D, int C, const float* w_head) {
  if (head_lds_bytes(D, C, w_head, TAKES_SCRATCH) > 64 * 1024) return false;
  return (int64_t)D * C < 300000 || (!four_classes(C, w_head) && B > 40);
}

void head_fwd_bwd(const void* x, int B, int Tl, int D, int C, bool f32, const float* gamma, const float* beta, float eps,
                  const float* w_head, const float* b_head, const int32_t* labels, float* xhat, float* z, float* logits,
                  float* dlogits, float* dz, float* loss_rows, void* dx, float* dw, float* db, float* dgamma, float* dbeta,
                  float* loss, hipStream_t s) {
  const size_t lds = head_lds_bytes(D, C, w_head, SCRATCH);          // (at most 68 KB)
  const dim3 grid(B, Tl > 1 ? 1 + ZERO_PARTS : 1);
  auto rows = [&](auto zero, auto vec, auto wide) {
    typedef decltype(zero) T;
    auto kern = head_rows_kernel<T, decltype(vec)::value, decltype(wide)::value != 0>;
    if (lds > 64 * 1024) (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    kern<<<grid, HT, lds, s>>>(
        (const T*)x, Tl, D, C, B, gamma, beta, eps, w_head, b_head, labels, xhat, z, logits, dlogits, dz, loss_rows, (T*)dx);
  };
  auto forms = [&](auto zero) {
    const bool wide = wide_head(C, w_head);
    if (four_classes(C, w_head)) wide ? rows(zero, RowC<4>{}, RowC<1>{}) : rows(zero, RowC<4>{}, RowC<0>{});
    else wide ? rows(zero, RowC<1>{}, RowC<1>{}) : rows(zero, RowC<1>{}, RowC<0>{});
  };
  if (f32) forms(0.f);
  else forms((bf16)0.f);
  const int nw = ((D + TD - 1) / TD) * ((C + TC - 1) / TC);
  head_batch_kernel<<<nw + (D + WAVE - 1) / WAVE + 1, BT, 0, s>>>(z, xhat, dlogits, dz, loss_rows, B, D, C, nw, dw, db, dgamma, dbeta,
                                                                loss);
}

}  // namespace bsr
