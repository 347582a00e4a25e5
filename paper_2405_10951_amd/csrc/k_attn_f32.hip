// fp32 softmax attention (Eq. 1) for head size 64, forward and backward, on the matrix cores
// (v_mfma_f32_32x32x2_f32): the attention of the fp32 mode, any number of tokens.
//
// What bounds it: the matrix cores (a 32 x 32 block of scores over 64 features is 32 MFMAs of 64 clocks, 2048 clocks),
// and at the sizes of this mode the number of wavefronts: one wavefront per 32 queries walks all keys in a row, 12 us
// at 197 tokens.  So a workgroup owns 32 rows and its four wavefronts share the other side, block by block; what they
// find (maximum, sum, partial output) is put together through LDS in a fixed order.  Operands come straight from
// global memory (a head's rows are a few 10 KB and stay in L2): MFMA contracts over a dummy index, so MFMA j of a
// group of 8 features uses feature 4 h + j for wave half h and a lane reads four consecutive floats; and the
// accumulator of the scores, whose element r holds row 8 (r / 4) + 4 h + r % 4, is itself the operand of the second
// product, with the other operand read in that row order.
// 8 images of 6 heads at 197 .. 67 tokens: forward 53 -> 12 us on average, backward 72 -> 18 us, against one wavefront
// per row on the vector unit.
#include "rowops.h"

namespace bsr {

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int HD = 64, NW = 4;          // head size, wavefronts per workgroup
constexpr int MAX_T = 1024;

__device__ inline int row_of(int r, int lh) { return 8 * (r >> 2) + 4 * lh + (r & 3); }
__device__ inline void zero(f32x16& a) {
#pragma unroll
  for (int r = 0; r < 16; ++r) a[r] = 0.f;
}
// this lane's half of a row: features 8 g + 4 h .. + 3
__device__ inline void load_row(const float* row, int lh, f32x4 (&f)[8]) {
#pragma unroll
  for (int g = 0; g < 8; ++g) f[g] = *(const f32x4*)(row + 8 * g + 4 * lh);
}
// acc[i, j] = sum over features of a_i b_j for 32 rows a (lane % 32) and 32 rows b (lane % 32)
__device__ inline f32x16 row_products(const f32x4 (&a)[8], const f32x4 (&b)[8]) {
  f32x16 acc;
  zero(acc);
#pragma unroll
  for (int g = 0; g < 8; ++g)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[g][j], b[g][j], acc, 0, 0, 0);
  return acc;
}

__global__ __launch_bounds__(NW * 64) void attn_f32_fwd_kernel(const float* __restrict__ qkv, int T, int H, float* __restrict__ out,
                                                              float* __restrict__ lse, float* __restrict__ cls_prob) {
  __shared__ float mls[NW][2][32];
  __shared__ float os[NW][2][16][64];
  __shared__ float cls_s[MAX_T];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lr = lane & 31, lh = lane >> 5;
  const int b = blockIdx.y / H, h = blockIdx.y % H, D = H * HD, q0 = blockIdx.x * 32;
  const int64_t rs = 3 * (int64_t)D;
  const float* base = qkv + (int64_t)b * T * rs + h * HD;
  const int qi = q0 + lr;
  const bool want_cls = cls_prob && q0 == 0;                   // uniform over the workgroup
  f32x4 qf[8];
  load_row(base + (int64_t)min(qi, T - 1) * rs, lh, qf);
  f32x16 o[2];
  zero(o[0]);
  zero(o[1]);
  float m = -INFINITY, l = 0.f;
  for (int k0 = wave * 32; k0 < T; k0 += NW * 32) {
    f32x4 kf[8];
    load_row(base + D + (int64_t)min(k0 + lr, T - 1) * rs, lh, kf);
    f32x16 s = row_products(kf, qf);                           // S^T: row = key, column (lane) = query
    float mx = m;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int key = k0 + row_of(r, lh);
      s[r] = key < T ? s[r] * 0.125f : -INFINITY;
      if (want_cls && lr == 0 && key < T) cls_s[key] = s[r];
      mx = fmaxf(mx, s[r]);
    }
    mx = half_max(mx);                    // finite: a block holds at least one key
    const float alpha = expf(m - mx);
    m = mx;
    float sum = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) { s[r] = expf(s[r] - mx); sum += s[r]; }
    l = l * alpha + sum + half_other(sum);
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) {
#pragma unroll
      for (int r = 0; r < 16; ++r) o[nb][r] *= alpha;
#pragma unroll
      for (int r = 0; r < 16; ++r) {                           // O^T += V^T P^T: row = feature, lane = query
        const float v = base[2 * D + (int64_t)min(k0 + row_of(r, lh), T - 1) * rs + nb * 32 + lr];
        o[nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(v, s[r], o[nb], 0, 0, 0);
      }
    }
  }
  if (lh == 0) { mls[wave][0][lr] = m; mls[wave][1][lr] = l; }
  __syncthreads();
  float mt = mls[0][0][lr];
#pragma unroll
  for (int w = 1; w < NW; ++w) mt = fmaxf(mt, mls[w][0][lr]);
  float lt = 0.f;
#pragma unroll
  for (int w = 0; w < NW; ++w) lt += mls[w][1][lr] * expf(mls[w][0][lr] - mt);
  const float own = expf(m - mt);                              // 0 for a wavefront without keys
#pragma unroll
  for (int nb = 0; nb < 2; ++nb)
#pragma unroll
    for (int r = 0; r < 16; ++r) os[wave][nb][r][lane] = o[nb][r] * own;
  __syncthreads();
  const float inv = 1.0f / lt;
  if (qi < T) {                                                // wavefront w finishes 16 of the 64 features
    const int nb = wave >> 1;
    float* orow = out + ((int64_t)b * T + qi) * D + h * HD + nb * 32 + 4 * lh;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int rq = (wave & 1) * 2 + q;
      f32x4 v;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float a = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) a += os[w][nb][4 * rq + e][lane];
        v[e] = a * inv;
      }
      *(f32x4*)(orow + 8 * rq) = v;
    }
    if (lse && wave == 0 && lh == 0) lse[((int64_t)b * H + h) * T + qi] = mt + logf(lt);
  }
  if (want_cls) {                                              // query 0 is lane 0 of either half
    const float m0 = __shfl(mt, 0, 64), i0 = __shfl(inv, 0, 64);
    for (int j = threadIdx.x; j < T; j += NW * 64) cls_prob[((int64_t)b * H + h) * T + j] = expf(cls_s[j] - m0) * i0;
  }
}

// adds the four wavefronts' 32 x 64 blocks in order and stores them: rows first .. of dst (row stride rs)
__device__ inline void reduce_store(const f32x16 (&o)[2], float (*os)[2][16][64], float* dst, int64_t rs, int first, int T, int wave,
                                    int lane) {
  const int lr = lane & 31, lh = lane >> 5;
  __syncthreads();
#pragma unroll
  for (int nb = 0; nb < 2; ++nb)
#pragma unroll
    for (int r = 0; r < 16; ++r) os[wave][nb][r][lane] = o[nb][r];
  __syncthreads();
  const int nb = wave >> 1;
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    const int r = (wave & 1) * 8 + q, i = first + row_of(r, lh);
    float a = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) a += os[w][nb][r][lane];
    if (i < T) dst[(int64_t)i * rs + nb * 32 + lr] = a;
  }
}

// the 32 x 64 operand of the second product as its MFMAs take it: row row_of(r), feature 32 nb + lane % 32
__device__ __forceinline__ void load_rows_t(const float* base, int64_t rs, int r0, int T, int lr, int lh, float (&v)[2][16]) {
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const float* row = base + (int64_t)min(r0 + row_of(r, lh), T - 1) * rs + lr;
    v[0][r] = row[0];
    v[1][r] = row[32];
  }
}

// Backward (Eq. 3, 5): P = exp(s / 8 - lse), dP = dO . v, delta = dO . O, dS = P (dP - delta) / 8.
// Workgroups [0, nb): dQ of 32 queries, the wavefronts share the keys; [nb, 2 nb): dK and dV of 32 keys, the
// wavefronts share the queries (delta is taken again from rows they read anyway, so both run in one launch).
// Bound by the wait for a block's rows before each of its products: the operands of all four are asked for ahead of
// the first that needs them, so one wait is left per block.  8 images of 6 heads, 197 tokens and the selected ones
// after them, three launches: 70 -> 53 us; 2 images of 3 heads at 65 tokens: 15.1 -> 12.7 us.
__global__ __launch_bounds__(NW * 64, 2) void attn_f32_bwd_kernel(const float* __restrict__ qkv, const float* __restrict__ out,
                                                              const float* __restrict__ dout, const float* __restrict__ lse, int T,
                                                              int H, float* __restrict__ dqkv) {
  __shared__ float os[NW][2][16][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lr = lane & 31, lh = lane >> 5;
  const int b = blockIdx.y / H, h = blockIdx.y % H, D = H * HD, nblk = (T + 31) / 32;
  const int64_t rs = 3 * (int64_t)D;
  const float* base = qkv + (int64_t)b * T * rs + h * HD;
  const float* obase = out + (int64_t)b * T * D + h * HD;
  const float* dobase = dout + (int64_t)b * T * D + h * HD;
  const float* lrow = lse + ((int64_t)b * H + h) * T;
  float* dbase = dqkv + (int64_t)b * T * rs + h * HD;
  auto delta_of = [&](int row, const f32x4 (&dof)[8]) {        // dO . O of that row, in both halves
    f32x4 of[8];
    load_row(obase + (int64_t)row * D, lh, of);
    float d = 0.f;
#pragma unroll
    for (int g = 0; g < 8; ++g)
#pragma unroll
      for (int e = 0; e < 4; ++e) d = fmaf(dof[g][e], of[g][e], d);
    return half_sum(d);
  };
  if ((int)blockIdx.x < nblk) {
    const int q0 = blockIdx.x * 32, qc = min(q0 + lr, T - 1);
    f32x4 qf[8], dof[8];
    load_row(base + (int64_t)qc * rs, lh, qf);
    load_row(dobase + (int64_t)qc * D, lh, dof);
    const float dl = delta_of(qc, dof), ls = lrow[qc];
    f32x16 o[2];
    zero(o[0]);
    zero(o[1]);
    for (int k0 = wave * 32; k0 < T; k0 += NW * 32) {
      const float* krow = base + D + (int64_t)min(k0 + lr, T - 1) * rs;
      f32x4 f[8], f2[8];
      load_row(krow, lh, f);
      load_row(krow + D, lh, f2);
      f32x16 s = row_products(f, qf);                          // row = key, lane = query
      float kt[2][16];                                         // on its way while dP is multiplied
      load_rows_t(base + D, rs, k0, T, lr, lh, kt);
      const f32x16 dp = row_products(f2, dof);
#pragma unroll
      for (int r = 0; r < 16; ++r)
        s[r] = k0 + row_of(r, lh) < T ? expf(s[r] * 0.125f - ls) * (dp[r] - dl) * 0.125f : 0.f;
#pragma unroll
      for (int nb = 0; nb < 2; ++nb)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          o[nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(s[r], kt[nb][r], o[nb], 0, 0, 0);      // row = query, lane = feature
    }
    reduce_store(o, os, dbase, rs, q0, T, wave, lane);
    return;
  }
  const int j0 = (blockIdx.x - nblk) * 32, jc = min(j0 + lr, T - 1);
  f32x4 kf[8], vf[8];
  load_row(base + D + (int64_t)jc * rs, lh, kf);
  load_row(base + 2 * D + (int64_t)jc * rs, lh, vf);
  f32x16 ok[2], ov[2];
  zero(ok[0]); zero(ok[1]); zero(ov[0]); zero(ov[1]);
  for (int i0 = wave * 32; i0 < T; i0 += NW * 32) {
    const int ic = min(i0 + lr, T - 1);
    f32x4 f[8], f2[8];
    load_row(base + (int64_t)ic * rs, lh, f);
    load_row(dobase + (int64_t)ic * D, lh, f2);
    f32x16 s = row_products(f, kf);                            // row = query, lane = key
    const float dl = delta_of(ic, f2), ls = lrow[ic];
    f32x16 dp = row_products(f2, vf);
    float gt[2][16], qt[2][16];                                // dO and Q as the second products take them
    load_rows_t(dobase, D, i0, T, lr, lh, gt);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int i = row_of(r, lh);
      const float li = __shfl(ls, i, 64), di = __shfl(dl, i, 64);
      const float p = i0 + i < T ? expf(s[r] * 0.125f - li) : 0.f;
      s[r] = p;
      dp[r] = p * (dp[r] - di) * 0.125f;
    }
    load_rows_t(base, rs, i0, T, lr, lh, qt);
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        ov[nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(s[r], gt[nb][r], ov[nb], 0, 0, 0);
        ok[nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(dp[r], qt[nb][r], ok[nb], 0, 0, 0);
      }
  }
  reduce_store(ok, os, dbase + D, rs, j0, T, wave, lane);
  reduce_store(ov, os, dbase + 2 * D, rs, j0, T, wave, lane);
}

}  // namespace

bool attn_f32_supported(int T, int d) { return d == HD && T >= 1 && T <= MAX_T; }

void attn_fwd_f32(const float* qkv, int B, int T, int H, float* out, float* lse, float* cls_prob, hipStream_t s) {
  attn_f32_fwd_kernel<<<dim3((T + 31) / 32, B * H), NW * 64, 0, s>>>(qkv, T, H, out, lse, cls_prob);
}

void attn_bwd_f32(const float* qkv, const float* out, const float* dout, const float* lse, int B, int T, int H, float* dqkv,
                  hipStream_t s) {
  attn_f32_bwd_kernel<<<dim3(2 * ((T + 31) / 32), B * H), NW * 64, 0, s>>>(qkv, out, dout, lse, T, H, dqkv);
}

}  // namespace bsr
