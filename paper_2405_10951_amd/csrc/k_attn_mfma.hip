// bf16 MFMA softmax attention (Eq. 1 of the paper) for head size 64 and up to 1024 tokens: up to 256 tokens (every
// ViT-B/16 and DeiT-S block at 224 pixels) a head's keys are staged whole and probabilities are bf16 factors of the second
// product, beyond that keys come in chunks and probabilities stay in fp32 (second half of the file).  The CLS row of the
// softmax map, which Eq. 6 ranks tokens by, leaves the forward kernel in fp32 as a by-product.
//
// Forward.  One workgroup = one (image, head), or half the queries of one (fwd_parts): K and V of the head are staged
// in one go, and each of its wavefronts owns 32 queries.  K and V sit in LDS row-major (swizzled 16-byte chunks);
// V^T fragments come from the LDS transpose read.  The wave computes S^T = K Q^T with 32x32x16 MFMAs, so that a
// lane owns one query and the softmax reductions over keys are in-register (plus one exchange between
// the two halves of the wave).  The normalised P^T accumulators are, as they lie in registers, an
// operand of the second product O^T = V^T P^T: MFMA contracts over a dummy index, so the key order
// that the accumulator layout dictates is simply applied to the V^T reads as well.  No T x T tensor
// ever leaves registers.
#include <climits>

#include "rowops.h"

namespace bsr {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));

constexpr int HD = 64;          // head size

// Chunk permutation of a row of 8 16-byte chunks (128 B, two rows per sweep of the 64 banks): chunk kc of
// row r sits at kc ^ swz(r).  It serves two access patterns without bank conflicts:
//   - row fragments (16 consecutive rows read the same logical chunk): the 8 rows of either parity get 8
//     different positions;
//   - transposed fragments (4 consecutive rows r..r+3, r % 4 == 0, 64 bytes each): bit 2 differs between
//     rows r and r+2 (and r+1, r+3), so the four rows hit the four 64-byte bank groups.
__device__ inline int swz(int row) { return (((row >> 1) & 1) << 2) | ((row >> 2) & 3); }

// key index of accumulator element r (of key block jb) held by a lane of wave half lh
__device__ inline int key_of(int jb, int r, int lh) { return jb * 32 + 8 * (r >> 2) + 4 * lh + (r & 3); }

// Rows [T,64] of one operand of one head -> LDS chunks; rows >= T are zero.
__device__ inline void load_one(const bf16* base, int64_t row_stride, int T, int Tpad, u32x4* Ks, int tid, int nthreads) {
  const int total = Tpad * 8;
  for (int c0 = tid; c0 < total; c0 += 4 * nthreads) {
    u32x4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int c = c0 + u * nthreads, row = c >> 3, kc = c & 7;
      v[u] = u32x4{0u, 0u, 0u, 0u};
      if (c < total && row < T) v[u] = *(const u32x4*)(base + (int64_t)row * row_stride + kc * 8);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int c = c0 + u * nthreads, row = c >> 3, kc = c & 7;
      if (c < total) Ks[row * 8 + (kc ^ swz(row))] = v[u];
    }
  }
}
// K and V of one head together
__device__ inline void load_two(const bf16* x, int64_t xs, const bf16* y, int64_t ys, int T, int Tpad, u32x4* Xs, u32x4* Ys, int tid,
                                int nthreads) {
  // four loads of either operand in flight per thread before the first LDS write: one trip to memory
  const int total = Tpad * 8;
  for (int c0 = tid; c0 < total; c0 += 4 * nthreads) {
    u32x4 v[4], w[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int c = c0 + u * nthreads, row = c >> 3, kc = c & 7;
      v[u] = w[u] = u32x4{0u, 0u, 0u, 0u};
      if (c < total && row < T) {
        v[u] = *(const u32x4*)(x + (int64_t)row * xs + kc * 8);
        w[u] = *(const u32x4*)(y + (int64_t)row * ys + kc * 8);
      }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int c = c0 + u * nthreads, row = c >> 3, kc = c & 7;
      if (c < total) {
        Xs[row * 8 + (kc ^ swz(row))] = v[u];
        Ys[row * 8 + (kc ^ swz(row))] = w[u];
      }
    }
  }
}

// Transposed fragment of a row-major LDS tile [rows][64 features] for the 32 features nb*32 .. +31:
// lane (feature nb*32 + lane % 32, half lh = lane / 32) receives rows 16 st + 4 lh + {0..3} and
// 16 st + 8 + 4 lh + {0..3}, the order in which a 32x32 accumulator holds its rows.  Two LDS
// transpose reads (ds_read_b64_tr_b16): within 16 lanes, lane 4e+q passes the address of 4 features of
// row e and lane j receives feature j of the four rows.
// (last: rows past it are read as that row)
__device__ inline bf16x8 lds_frag_t(const u32x4* rows, int nb, int lane, int st, int last = INT_MAX) {
  const int j = lane & 15, cb = (lane >> 4) & 1, lh = lane >> 5;
  const int chunk = nb * 4 + cb * 2 + ((j & 3) >> 1), half = j & 1;
  const int r0 = min(16 * st + 4 * lh + (j >> 2), last), r1 = min(16 * st + 4 * lh + (j >> 2) + 8, last);
  const unsigned char* p = (const unsigned char*)rows;
  union { bf16x8 v; s16x4 h[2]; } f;
  f.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (s16x4 __attribute__((address_space(3)))*)(p + (r0 * 8 + (chunk ^ swz(r0))) * 16 + half * 8));
  f.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (s16x4 __attribute__((address_space(3)))*)(p + (r1 * 8 + (chunk ^ swz(r1))) * 16 + half * 8));
  return f.v;
}

// Rows of K and V in LDS: the tokens and at least one row of zeros where the last block of 32 has room for it, which stands for all rows past it.
__host__ __device__ inline int fwd_rows(int nj, int T) { return min(nj * 32, (T + 8) & ~7); }
// Workgroups that a head's queries go to; with two, both stage K and V.  What bounds the kernel is the softmax arithmetic and how many wavefronts a CU has to cover it.
// Kernel times, whole heads -> halves:
//   up to 128 heads leave CUs idle: one image of 12 heads at 197 tokens 8.0 -> 7.4 us.
//   129 .. 256 heads are one round of whole heads over the CUs, and halves would be more than one a CU: 132 heads 7.4 -> 7.9 us at 161 tokens, 8.2 -> 8.4 at 197, 8.3 -> 8.5 at 211;
//     252 8.2 -> 9.1, 9.2 -> 9.9 and 9.3 -> 10.3; 256 9.2 -> 9.5 at 211 (all of 161 .. 224 tokens and 132 .. 256 heads tried 1.02 .. 1.16).  Up to 160 tokens whole heads at any more heads.
//   161 .. 199 tokens, more heads: of whole heads a CU holds one of seven wavefronts (168 registers: three a SIMD) or two of six, of halves three, with up to 200 rows
//     staged, 52 KB: finer shares of the work, and beyond 192 tokens half as many wavefronts again.  258 heads 13.0 -> 10.2 at 161 tokens, 15.0 -> 11.6 at 197; 288 13.1 -> 10.1
//     and 15.2 -> 11.3; 384 13.4 -> 10.4 and 15.8 -> 12.3; 1536 41.9 -> 41.4 and 50.9 -> 49.8.
//   200 .. 224 tokens (208 rows of 256 bytes and the class row are 54 144: the CU's 160 KB are given out in steps that hold two): the same seven wavefronts
//     at work either way, but two workgroups that do not wait for each other, and K and V twice.  Up to 1.5 rounds of the CUs halves gain: 288 heads 15.5 -> 14.2
//     at 211 tokens, 384 16.7 -> 15.8 (258, the first of them, 15.1 -> 15.4).  Beyond, the second K and V cost more: 432 17.5 -> 17.8, 504 19.6 -> 20.4, 768 28.3 -> 31.6, 960 34.6 -> 38.2, 1536 50.8 -> 54.8
//     (where a last round of CUs is nearly empty the other way: 1284 50.0 -> 48.7), until qkv and output together outgrow the last-level cache and the kernel
//     waits for memory: 2556 heads at 200 tokens (262 MB) 80.6 -> 83.8, 2688 90.9 -> 89.4, 2880 106.8 -> 98.9; 2304 at 224 (264 MB) 79.9 -> 79.9, 2556 97.4 -> 95.5.
__host__ __device__ constexpr bool fwd_halves(int nj) { return nj == 6 || nj == 7; }      // forms that are held to three wavefronts a SIMD for it
inline int fwd_parts(int nj, int T, int64_t heads) {
  if (nj == 1) return 1;
  if (heads <= 128) return 2;
  if (!fwd_halves(nj) || heads <= 256) return 1;
  return fwd_rows(nj, T) <= 200 || heads <= 416 || heads * T * 4 * HD * (int64_t)sizeof(bf16) > (int64_t)256 << 20 ? 2 : 1;
}

// (97 .. 128 tokens are held to three wavefronts a SIMD as well: left alone that form takes 108 registers and 64 for accumulators beside them, held 117 in all, and
// four wavefronts fit.  384 heads at 97 tokens 8.5 -> 6.9 us, at 128 9.2 -> 7.8, 1536 heads 21.5 -> 18.1 and 24.4 -> 20.8.)
template <int NJ>
__global__ __launch_bounds__(NJ * 64, NJ == 4 || fwd_halves(NJ) ? 3 : 1) void attn_fwd_mfma_kernel(const bf16* __restrict__ qkv, int T, int H,
                                                               bf16* __restrict__ out, float* __restrict__ lse,
                                                               float* __restrict__ cls_prob) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int rows = fwd_rows(NJ, T);
  u32x4* Ks = (u32x4*)smem;                         // [rows][8 chunks]
  u32x4* Vs = Ks + rows * 8;                        // [rows][8 chunks]
  float* cls_s = (float*)(Vs + rows * 8);           // [32 NJ]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lr = lane & 31, lh = lane >> 5;
  const int b = blockIdx.x / H, h = blockIdx.x % H;
  const int D = H * HD;
  const int64_t rs = 3 * (int64_t)D;
  const bf16* base = qkv + (int64_t)b * T * rs + h * HD;
  const int q0 = (blockIdx.y * (blockDim.x >> 6) + wave) * 32;      // a wave owns 32 queries
  // Q fragments straight from global memory, requested before K and V are staged so that their
  // latency is hidden: lane (query lr, half lh) needs chunks 2 ks + lh
  bf16x8 qf[4];
  {
    const bf16* qrow = base + (int64_t)min(q0 + lr, T - 1) * rs;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) qf[ks] = *(const bf16x8*)(qrow + (2 * ks + lh) * 8);
  }
  load_two(base + D, rs, base + 2 * D, rs, T, rows, Ks, Vs, tid, blockDim.x);
  __syncthreads();
  if (q0 >= T) return;

  // S^T[key, query] = K Q^T
  f32x16 s[NJ];
  const int sw = swz(lr);
#pragma unroll
  for (int jb = 0; jb < NJ; ++jb) {
#pragma unroll
    for (int r = 0; r < 16; ++r) s[jb][r] = 0.f;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      const int row = jb == NJ - 1 ? min(jb * 32 + lr, rows - 1) : jb * 32 + lr;
      const bf16x8 kf = *(const bf16x8*)(Ks + row * 8 + ((2 * ks + lh) ^ (jb == NJ - 1 ? swz(row) : sw)));
      s[jb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[ks], s[jb], 0, 0, 0);
    }
  }
  // softmax over keys: this lane holds, for query q0 + lr, the keys key_of(jb, r, lh).  The probabilities
  // stay unnormalised (p = exp(s - max) in (0, 1]) on their way through the second product; 1 / sum is
  // applied to the 32 output values instead of the 32 NJ probabilities.
  const float c = 0.125f * 1.44269504088896341f;    // 1/sqrt(64) * log2(e)
  float mx = -INFINITY;
#pragma unroll
  for (int jb = 0; jb < NJ; ++jb) {
    if (jb * 32 + 32 > T) {                         // only the last key block can hold keys past T (uniform)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (key_of(jb, r, lh) >= T) s[jb][r] = -INFINITY;
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[jb][r]);
  }
  mx = half_max(mx);
  const float mc = mx * c;
  float sum = 0.f;
  bf16x8 pf[2 * NJ];
#pragma unroll
  for (int jb = 0; jb < NJ; ++jb)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float p = __builtin_amdgcn_exp2f(fmaf(s[jb][r], c, -mc));
      s[jb][r] = p;
      sum += p;
      pf[2 * jb + (r >> 3)][r & 7] = (bf16)p;
    }
  sum = half_sum(sum);
  const float inv = 1.0f / sum;
  const int qi = q0 + lr;
  if (lse && lh == 0 && qi < T) lse[((int64_t)b * H + h) * T + qi] = mx * 0.125f + __logf(sum);
  if (cls_prob && q0 == 0) {   // the wavefront of the CLS query: its softmax row in fp32 (Eq. 6), through LDS to leave in whole rows
    if (lr == 0)
#pragma unroll
      for (int jb = 0; jb < NJ; ++jb)
#pragma unroll
        for (int r = 0; r < 16; r += 4)
          *(float4*)(cls_s + key_of(jb, r, lh)) = make_float4(s[jb][r] * inv, s[jb][r + 1] * inv, s[jb][r + 2] * inv, s[jb][r + 3] * inv);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    float* dst = cls_prob + ((int64_t)b * H + h) * T;
    for (int j = lane; j < T; j += 64) dst[j] = cls_s[j];
  }
  // O^T = V^T P^T, contraction over keys in the order the accumulators hold them:
  // step st covers keys 16 st + {4 lh .. 4 lh + 3} and 16 st + 8 + {4 lh .. 4 lh + 3}.
  // With the features as rows, a lane ends up with 4 consecutive features of its own query per
  // accumulator quad: the output leaves in 8-byte stores.
  f32x16 o[2];
#pragma unroll
  for (int nb = 0; nb < 2; ++nb) {
#pragma unroll
    for (int r = 0; r < 16; ++r) o[nb][r] = 0.f;
#pragma unroll
    for (int st = 0; st < 2 * NJ; ++st)
      o[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lds_frag_t(Vs, nb, lane, st, st >= 2 * NJ - 2 ? rows - 1 : INT_MAX), pf[st], o[nb], 0, 0, 0);
  }
  if (qi < T) {
    bf16* orow = out + ((int64_t)b * T + qi) * D + h * HD + 4 * lh;
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
      for (int rq = 0; rq < 4; ++rq) {
        bf16x4 v4;
#pragma unroll
        for (int e = 0; e < 4; ++e) v4[e] = (bf16)(o[nb][4 * rq + e] * inv);
        *(bf16x4*)(orow + nb * 32 + 8 * rq) = v4;
      }
  }
}

template <int NJ>
void launch_fwd(const bf16* qkv, int B, int T, int H, bf16* out, float* lse, float* cls_prob, hipStream_t s) {
  static bool attr_set = false;
  const auto lds = [](int rows) { return (size_t)2 * rows * 128 + NJ * 32 * sizeof(float); };
  if (!attr_set) {
    (void)hipFuncSetAttribute((const void*)attn_fwd_mfma_kernel<NJ>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds(NJ * 32));
    attr_set = true;
  }
  const int parts = fwd_parts(NJ, T, (int64_t)B * H);
  attn_fwd_mfma_kernel<NJ><<<dim3(B * H, parts), (NJ + parts - 1) / parts * 64, lds(fwd_rows(NJ, T)), s>>>(qkv, T, H, out, lse, cls_prob);
}


// ------------------------------------------------------------------------------------------ backward
// Backward of Eq. 1 per head (the "non-linear layer" case of Eq. 3 / Eq. 5: it needs the stored
// q, k, v and the softmax statistics).  With P_ij = exp(s_ij / 8 - lse_i), dP_ij = dO_i . v_j,
// delta_i = dO_i . O_i (= sum_j P_ij dP_ij) and dS_ij = P_ij (dP_ij - delta_i) / 8:
//   dQ_i = sum_j dS_ij k_j      (kernel "dq":  a wave owns 32 queries, sweeps the key blocks)
//   dK_j = sum_i dS_ij q_i,  dV_j = sum_i P_ij dO_i   (kernel "dkv": a wave owns 32 keys, sweeps
//                                                      the query blocks)
// These two are for 225 .. 256 tokens, whose score gradients do not fit in LDS beside the operands (below: attn_bwd_kernel).
// Both recompute S with MFMAs; nothing T x T is stored or exchanged between wavefronts, and no
// atomics are used.  What bounds them is how many wavefronts a CU has to cover the chain read - MFMA - exp - MFMA.  "dq" runs all
// ceil(T / 32) wavefronts of a head in one workgroup, in 128 registers, so that two heads share a CU, and writes 8-byte pieces:
// 128 images of 12 heads at 197 tokens 89 -> 67 us (four wavefronts a workgroup, a head staged twice, 2-byte stores).  "dkv" has
// four accumulators and needs 124 registers with its loop written out; held to 128 in workgroups of seven wavefronts it spills
// (135 us), with the loop kept it takes 108, and 8-byte stores alone make it 93: so it stays at 84.  As in the forward kernel the lane that owns the output row keeps the
// contraction index in accumulator order and the transposed operand in LDS is read in that order.

__device__ inline bf16x8 lds_frag(const u32x4* rows, int row, int chunk) {
  return *(const bf16x8*)(rows + row * 8 + (chunk ^ swz(row)));
}

// 64 features of one row, features as rows of the accumulators, lane = row
__device__ __forceinline__ void store_row(bf16* row, const f32x16 (&o)[2], int lh) {
#pragma unroll
  for (int nb = 0; nb < 2; ++nb)
#pragma unroll
    for (int rq = 0; rq < 4; ++rq) {
      bf16x4 v4;
#pragma unroll
      for (int e = 0; e < 4; ++e) v4[e] = (bf16)o[nb][4 * rq + e];
      *(bf16x4*)(row + nb * 32 + 8 * rq + 4 * lh) = v4;
    }
}

template <int NJ>
__global__ __launch_bounds__(NJ * 64, 4) void attn_bwd_dq_kernel(const bf16* __restrict__ qkv, const bf16* __restrict__ out,
                                                          const bf16* __restrict__ dout, const float* __restrict__ lse,
                                                          int T, int H, float* __restrict__ delta,
                                                          bf16* __restrict__ dqkv) {
  constexpr int Tpad = NJ * 32;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  u32x4* Ks = (u32x4*)smem;
  u32x4* Vs = Ks + Tpad * 8;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lr = lane & 31, lh = lane >> 5;
  const int b = blockIdx.x / H, h = blockIdx.x % H;
  const int D = H * HD;
  const int64_t rs = 3 * (int64_t)D;
  const bf16* base = qkv + (int64_t)b * T * rs + h * HD;
  load_two(base + D, rs, base + 2 * D, rs, T, Tpad, Ks, Vs, tid, NJ * 64);
  __syncthreads();
  const int q0 = wave * 32;
  const int qi = q0 + lr, qc = min(qi, T - 1);
  bf16x8 qf[4], dof[4];
  float dl = 0.f;
  {
    const bf16* qrow = base + (int64_t)qc * rs;
    const bf16* dorow = dout + ((int64_t)b * T + qc) * D + h * HD;
    const bf16* orow = out + ((int64_t)b * T + qc) * D + h * HD;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      qf[ks] = *(const bf16x8*)(qrow + (2 * ks + lh) * 8);
      dof[ks] = *(const bf16x8*)(dorow + (2 * ks + lh) * 8);
      const bf16x8 of = *(const bf16x8*)(orow + (2 * ks + lh) * 8);
#pragma unroll
      for (int e = 0; e < 8; ++e) dl += (float)dof[ks][e] * (float)of[e];
    }
  }
  dl = half_sum(dl);
  const float l2 = lse[((int64_t)b * H + h) * T + qc] * 1.44269504088896341f;
  if (lh == 0 && qi < T) delta[((int64_t)b * H + h) * T + qi] = dl;
  const float c = 0.125f * 1.44269504088896341f;
  f32x16 o[2];
#pragma unroll
  for (int nb = 0; nb < 2; ++nb)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[nb][r] = 0.f;
#pragma nounroll
  for (int jb = 0; jb < NJ; ++jb) {
    f32x16 sa, dp;
#pragma unroll
    for (int r = 0; r < 16; ++r) { sa[r] = 0.f; dp[r] = 0.f; }
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      sa = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lds_frag(Ks, jb * 32 + lr, 2 * ks + lh), qf[ks], sa, 0, 0, 0);
      dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lds_frag(Vs, jb * 32 + lr, 2 * ks + lh), dof[ks], dp, 0, 0, 0);
    }
    bf16x8 dsf[2];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      float pr = __builtin_amdgcn_exp2f(sa[r] * c - l2);
      if (jb == NJ - 1 && key_of(jb, r, lh) >= T) pr = 0.f;
      dsf[r >> 3][r & 7] = (bf16)(pr * (dp[r] - dl) * 0.125f);
    }
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
      for (int hf = 0; hf < 2; ++hf)
        o[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lds_frag_t(Ks, nb, lane, 2 * jb + hf), dsf[hf], o[nb], 0, 0, 0);
  }
  if (qi < T) store_row(dqkv + ((int64_t)b * T + qi) * rs + h * HD, o, lh);
}

template <int NJ>
__global__ __launch_bounds__(256) void attn_bwd_dkv_kernel(const bf16* __restrict__ qkv, const bf16* __restrict__ dout,
                                                           const float* __restrict__ lse, const float* __restrict__ delta,
                                                           int T, int H, bf16* __restrict__ dqkv) {
  constexpr int Tpad = NJ * 32;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  u32x4* Qs = (u32x4*)smem;
  u32x4* dOs = Qs + Tpad * 8;
  float* lse_s = (float*)(dOs + Tpad * 8);      // [Tpad], pre-multiplied by log2(e); +inf beyond T
  float* del_s = lse_s + Tpad;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lr = lane & 31, lh = lane >> 5;
  const int b = blockIdx.y / H, h = blockIdx.y % H;
  const int D = H * HD;
  const int64_t rs = 3 * (int64_t)D;
  const bf16* base = qkv + (int64_t)b * T * rs + h * HD;
  const bf16* dobase = dout + (int64_t)b * T * D + h * HD;
  load_one(base, rs, T, Tpad, Qs, tid, 256);        // (both at once: registers that this kernel needs, 84 -> 88 us)
  load_one(dobase, D, T, Tpad, dOs, tid, 256);
  for (int i = tid; i < Tpad; i += 256) {
    lse_s[i] = (i < T) ? lse[((int64_t)b * H + h) * T + i] * 1.44269504088896341f : INFINITY;
    del_s[i] = (i < T) ? delta[((int64_t)b * H + h) * T + i] : 0.f;
  }
  __syncthreads();
  const int j0 = blockIdx.x * 128 + wave * 32;
  if (j0 >= T) return;
  const int jc = min(j0 + lr, T - 1);
  bf16x8 kf[4], vf[4];
  {
    const bf16* krow = base + (int64_t)jc * rs + D;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      kf[ks] = *(const bf16x8*)(krow + (2 * ks + lh) * 8);
      vf[ks] = *(const bf16x8*)(krow + D + (2 * ks + lh) * 8);
    }
  }
  const float c = 0.125f * 1.44269504088896341f;
  f32x16 ok[2], ov[2];
#pragma unroll
  for (int nb = 0; nb < 2; ++nb)
#pragma unroll
    for (int r = 0; r < 16; ++r) { ok[nb][r] = 0.f; ov[nb][r] = 0.f; }
#pragma unroll
  for (int ib = 0; ib < NJ; ++ib) {
    f32x16 sa, dp;
#pragma unroll
    for (int r = 0; r < 16; ++r) { sa[r] = 0.f; dp[r] = 0.f; }
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      sa = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lds_frag(Qs, ib * 32 + lr, 2 * ks + lh), kf[ks], sa, 0, 0, 0);
      dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lds_frag(dOs, ib * 32 + lr, 2 * ks + lh), vf[ks], dp, 0, 0, 0);
    }
    bf16x8 pf[2], dsf[2];
#pragma unroll
    for (int g4 = 0; g4 < 4; ++g4) {           // queries 32 ib + 8 g4 + 4 lh + {0..3}
      const float4 l4 = *(const float4*)(lse_s + ib * 32 + 8 * g4 + 4 * lh);
      const float4 d4 = *(const float4*)(del_s + ib * 32 + 8 * g4 + 4 * lh);
      const float lv[4] = {l4.x, l4.y, l4.z, l4.w};
      const float dv[4] = {d4.x, d4.y, d4.z, d4.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int r = g4 * 4 + e;
        const float pr = __builtin_amdgcn_exp2f(sa[r] * c - lv[e]);
        pf[r >> 3][r & 7] = (bf16)pr;
        dsf[r >> 3][r & 7] = (bf16)(pr * (dp[r] - dv[e]) * 0.125f);
      }
    }
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
      for (int hf = 0; hf < 2; ++hf) {
        ov[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(pf[hf], lds_frag_t(dOs, nb, lane, 2 * ib + hf), ov[nb], 0, 0, 0);
        ok[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(dsf[hf], lds_frag_t(Qs, nb, lane, 2 * ib + hf), ok[nb], 0, 0, 0);
      }
  }
#pragma unroll
  for (int nb = 0; nb < 2; ++nb)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int j = j0 + 8 * (r >> 2) + 4 * lh + (r & 3);
      if (j < T) {
        bf16* dst = dqkv + ((int64_t)b * T + j) * rs + h * HD + nb * 32 + lr;
        dst[D] = (bf16)ok[nb][r];
        dst[2 * D] = (bf16)ov[nb][r];
      }
    }
}

// All three in one launch, up to 224 tokens.  A wavefront owns 32 keys and sweeps the query blocks as in "dkv"; the score gradients, which dQ
// needs with the keys as contraction index, stay in LDS (ceil(T / 32) blocks of [key][32 queries] in bf16, the factor that "dq" rounds them to), and
// once every wavefront is done each turns to 32 queries and contracts them with the keys, which by then lie where the queries were.  So scores,
// probabilities and dP are computed once instead of twice, q, k, v and dO are read once, and delta never leaves LDS but for the caller's copy.
// Same products in the same order: the same bits as the two kernels.  What bounds it at many images is
// memory (310 MB at 128 images of 12 heads and 197 tokens, 66 us of the 114), with one head a CU at a time.  Two kernels -> this: 128 images of 12 heads,
// 197 tokens 148 -> 114 us, 138 tokens 109 -> 79, 67 tokens 44 -> 32; 32 images 48 -> 35, 35 -> 25, 15.5 -> 11.3; one image 19.5 -> 15.0.
// dS rows are four 16-byte chunks, chunk c of key j at c ^ ((j >> 2) & 3): 8-byte writes of 32 keys and the transpose reads of 4 keys x 32
// queries touch every bank alike.
template <int NJ> constexpr size_t attn_bwd_lds() {
  return (size_t)2 * NJ * 32 * 128 + (size_t)NJ * NJ * 32 * 64 + (size_t)2 * NJ * 32 * sizeof(float);
}
template <int NJ>
__global__ __launch_bounds__(NJ * 64) void attn_bwd_kernel(const bf16* __restrict__ qkv, const bf16* __restrict__ out, const bf16* __restrict__ dout,
                                                           const float* __restrict__ lse, int T, int H, float* __restrict__ delta,
                                                           bf16* __restrict__ dqkv) {
  constexpr int Tpad = NJ * 32;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  u32x4* Qs = (u32x4*)smem;
  u32x4* dOs = Qs + Tpad * 8;
  unsigned char* dS = (unsigned char*)(dOs + Tpad * 8);      // [NJ query blocks][Tpad keys][64 bytes]
  float* lse_s = (float*)(dS + NJ * Tpad * 64);              // [Tpad], pre-multiplied by log2(e); +inf beyond T
  float* del_s = lse_s + Tpad;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 31, lh = lane >> 5;
  const int b = blockIdx.x / H, h = blockIdx.x % H;
  const int D = H * HD;
  const int64_t rs = 3 * (int64_t)D;
  const bf16* base = qkv + (int64_t)b * T * rs + h * HD;
  const bf16* dobase = dout + (int64_t)b * T * D + h * HD;
  const int j0 = wave * 32, ji = j0 + lr, jc = min(ji, T - 1);       // this lane's key, and later its query
  bf16x8 kf[4], vf[4];
  float dl = 0.f;
  {
    const bf16* krow = base + (int64_t)jc * rs + D;
    const bf16* dorow = dobase + (int64_t)jc * D;
    const bf16* orow = out + ((int64_t)b * T + jc) * D + h * HD;
    bf16x8 df[4], of[4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      df[ks] = *(const bf16x8*)(dorow + (2 * ks + lh) * 8);
      of[ks] = *(const bf16x8*)(orow + (2 * ks + lh) * 8);
      kf[ks] = *(const bf16x8*)(krow + (2 * ks + lh) * 8);
      vf[ks] = *(const bf16x8*)(krow + D + (2 * ks + lh) * 8);
    }
    load_two(base, rs, dobase, D, T, Tpad, Qs, dOs, tid, NJ * 64);
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
      for (int e = 0; e < 8; ++e) dl += (float)df[ks][e] * (float)of[ks][e];
  }
  dl = half_sum(dl);
  if (lh == 0) {
    const bool valid = ji < T;
    lse_s[ji] = valid ? lse[((int64_t)b * H + h) * T + ji] * 1.44269504088896341f : INFINITY;
    del_s[ji] = valid ? dl : 0.f;
    if (valid) delta[((int64_t)b * H + h) * T + ji] = dl;
  }
  __syncthreads();
  const float c = 0.125f * 1.44269504088896341f;
  f32x16 ok[2], ov[2];
#pragma unroll
  for (int nb = 0; nb < 2; ++nb)
#pragma unroll
    for (int r = 0; r < 16; ++r) { ok[nb][r] = 0.f; ov[nb][r] = 0.f; }
  // The scores of query block ib + 1 are under way in the matrix cores while block ib goes through its exponentials: a CU holds one head of
  // more than 128 tokens, 1 - 2 wavefronts a SIMD, and nobody else covers either
  // (197 tokens, 128 images: 118 -> 114 us).
  f32x16 sa, dp;
#pragma unroll
  for (int r = 0; r < 16; ++r) { sa[r] = 0.f; dp[r] = 0.f; }
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) {
    sa = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lds_frag(Qs, lr, 2 * ks + lh), kf[ks], sa, 0, 0, 0);
    dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lds_frag(dOs, lr, 2 * ks + lh), vf[ks], dp, 0, 0, 0);
  }
#pragma unroll
  for (int ib = 0; ib < NJ; ++ib) {
    f32x16 san, dpn;
    bf16x8 fq[4], fd[4];
#pragma unroll
    for (int r = 0; r < 16; ++r) { san[r] = 0.f; dpn[r] = 0.f; }
    if (ib + 1 < NJ) {
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        fq[ks] = lds_frag(Qs, (ib + 1) * 32 + lr, 2 * ks + lh);
        fd[ks] = lds_frag(dOs, (ib + 1) * 32 + lr, 2 * ks + lh);
      }
    }
    bf16x8 pf[2], dsf[2];
    unsigned char* row = dS + (ib * Tpad + ji) * 64;
#pragma unroll
    for (int g4 = 0; g4 < 4; ++g4) {           // queries 32 ib + 8 g4 + 4 lh + {0..3}
      if (ib + 1 < NJ) {
        san = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fq[g4], kf[g4], san, 0, 0, 0);
        dpn = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fd[g4], vf[g4], dpn, 0, 0, 0);
      }
      const float4 l4 = *(const float4*)(lse_s + ib * 32 + 8 * g4 + 4 * lh);
      const float4 d4 = *(const float4*)(del_s + ib * 32 + 8 * g4 + 4 * lh);
      const float lv[4] = {l4.x, l4.y, l4.z, l4.w};
      const float dv[4] = {d4.x, d4.y, d4.z, d4.w};
      bf16x4 q4;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int r = g4 * 4 + e;
        const float pr = __builtin_amdgcn_exp2f(sa[r] * c - lv[e]);
        const bf16 ds = (bf16)(pr * (dp[r] - dv[e]) * 0.125f);
        pf[r >> 3][r & 7] = (bf16)pr;
        dsf[r >> 3][r & 7] = ds;
        q4[e] = ji < T ? ds : (bf16)0.f;       // keys past the end repeat the last one: nothing of theirs in dQ
      }
      *(bf16x4*)(row + ((g4 ^ ((ji >> 2) & 3)) << 4) + lh * 8) = q4;
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
      for (int hf = 0; hf < 2; ++hf) {
        ov[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lds_frag_t(dOs, nb, lane, 2 * ib + hf), pf[hf], ov[nb], 0, 0, 0);
        ok[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lds_frag_t(Qs, nb, lane, 2 * ib + hf), dsf[hf], ok[nb], 0, 0, 0);
      }
    sa = san;
    dp = dpn;
  }
  if (ji < T) {
    store_row(dqkv + ((int64_t)b * T + ji) * rs + D + h * HD, ok, lh);
    store_row(dqkv + ((int64_t)b * T + ji) * rs + 2 * D + h * HD, ov, lh);
  }
  __syncthreads();                             // the queries have been read, every score gradient is there
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) *(bf16x8*)(Qs + ji * 8 + ((2 * ks + lh) ^ swz(ji))) = kf[ks];
  __syncthreads();
  f32x16 o[2];
#pragma unroll
  for (int nb = 0; nb < 2; ++nb)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[nb][r] = 0.f;
  // lane j of 16 (cb: which 16 queries) gets queries' column j of key rows r .. r + 3, as in lds_frag_t
  const int j = lane & 15, cb = (lane >> 4) & 1, chunk = cb * 2 + ((j & 3) >> 1), half = j & 1;
  const unsigned char* blk = dS + wave * Tpad * 64;
#pragma unroll
  for (int st = 0; st < 2 * NJ; ++st) {
    const int r0 = 16 * st + 4 * lh + (j >> 2), r1 = r0 + 8;
    union { bf16x8 v; s16x4 h[2]; } f;
    f.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (s16x4 __attribute__((address_space(3)))*)(blk + r0 * 64 + ((chunk ^ ((r0 >> 2) & 3)) << 4) + half * 8));
    f.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (s16x4 __attribute__((address_space(3)))*)(blk + r1 * 64 + ((chunk ^ ((r1 >> 2) & 3)) << 4) + half * 8));
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) o[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lds_frag_t(Qs, nb, lane, st), f.v, o[nb], 0, 0, 0);
  }
  if (ji < T) store_row(dqkv + ((int64_t)b * T + ji) * rs + h * HD, o, lh);
}

template <int NJ>
void launch_bwd_one(const bf16* qkv, const bf16* out, const bf16* dout, const float* lse, int B, int T, int H, float* delta, bf16* dqkv, hipStream_t s) {
  static bool attr_set = false;
  constexpr size_t lds = attn_bwd_lds<NJ>();
  static_assert(lds <= 160 * 1024, "a head's operands and score gradients fit a CU");
  if (!attr_set) {
    (void)hipFuncSetAttribute((const void*)attn_bwd_kernel<NJ>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    attr_set = true;
  }
  attn_bwd_kernel<NJ><<<B * H, NJ * 64, lds, s>>>(qkv, out, dout, lse, T, H, delta, dqkv);
}

template <int NJ>
void launch_bwd(const bf16* qkv, const bf16* out, const bf16* dout, const float* lse, int B, int T, int H,
                float* delta, bf16* dqkv, hipStream_t s) {
  static bool attr_set = false;
  constexpr size_t lds_q = (size_t)2 * NJ * 32 * 128;
  constexpr size_t lds_kv = (size_t)2 * NJ * 32 * 128 + (size_t)2 * NJ * 32 * sizeof(float);
  if (!attr_set) {
    (void)hipFuncSetAttribute((const void*)attn_bwd_dq_kernel<NJ>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_q);
    (void)hipFuncSetAttribute((const void*)attn_bwd_dkv_kernel<NJ>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_kv);
    attr_set = true;
  }
  const dim3 grid((T + 127) / 128, B * H);
  attn_bwd_dq_kernel<NJ><<<B * H, NJ * 64, lds_q, s>>>(qkv, out, dout, lse, T, H, delta, dqkv);
  attn_bwd_dkv_kernel<NJ><<<grid, 256, lds_kv, s>>>(qkv, dout, lse, delta, T, H, dqkv);
}

// ------------------------------------------------------------------------------------------ more than 256 tokens
// The same products with the other side of the softmax walked in chunks of LC rows that pass through LDS (fetched
// into registers while the previous chunk is worked on): a workgroup owns 128 queries (4 wavefronts of 32) and the
// softmax is kept running, output and sum rescaled when a chunk raises the maximum.  Probabilities, score gradients and
// delta stay in fp32 here (Split below), so results are the exact ones rounded to bf16.  What bounds it is the softmax
// arithmetic (VALU) beside 12 MFMAs per 32 x 32 scores and the registers of the accumulators: held to 256 (two workgroups per
// CU) the kernels run 1.4 times as fast as with the 284 the compiler takes by itself.  At 577 tokens, 16 images of 6 heads, calls
// in a loop: 25.7 us forward and 75 backward (732 and 2711 with one wavefront per query, of the same precision; 37 and 100 with
// bf16 factors at 1 workgroup per CU, dq and dk 1.4 to 2.6 times as far from the exact ones).  Blocks of 32 keys or queries past the last token
// are left out, and wavefronts without a query or key of their own only stage; that the blocks of a chunk then are separate pieces of code lets
// exponentials and MFMAs of neighbouring blocks mix, and takes 204 registers instead of 256 (with whole chunks written out without the branch 28.2):
// forward and backward 28.5 -> 25.7 and 80.7 -> 75 us at 577 tokens, 22.2 -> 19.1 and 58.8 -> 50.3 at 404, 16.3 -> 12.4 and 44.4 -> 36.9 at 283, 4 images of 785
// 30.5 -> 21.2 and 59.3 -> 55.4.  Where every chunk is whole (384 .. 1024 tokens) the forward takes 0.72 .. 0.94 times as long, the backward 0.99 .. 1.00 from 48 heads on;
// for fewer, a chain of dependent blocks, the branches cost it 0.2 .. 0.8 us of 23 .. 53.
// Workgroups are numbered head first: the query blocks of a head then run on one XCD and share its L2.
constexpr int LC = 128, LCB = LC / 32, LONG_T = 1024;

// An fp32 factor as the sum of two bf16 ones, good to 2^-17: the second products of these lengths take probabilities and
// score gradients in fp32, each as two MFMAs with the same other operand.
struct Split {
  bf16x8 hi, lo;
  __device__ __forceinline__ void set2(int i, float v, float w) {      // elements i, i + 1: conversions come in pairs
    const bf16x2 a = __builtin_convertvector(f32x2{v, w}, bf16x2);
    const bf16x2 b = __builtin_convertvector(f32x2{v - (float)a[0], w - (float)a[1]}, bf16x2);
    hi[i] = a[0]; hi[i + 1] = a[1];
    lo[i] = b[0]; lo[i + 1] = b[1];
  }
};

struct ChunkRegs { u32x4 v[4]; };      // a thread's share of one operand's chunk: LC rows of 8 16-byte pieces, 256 threads
__device__ inline void chunk_fetch(ChunkRegs& c, const bf16* base, int64_t rs, int r0, int T, int tid) {
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int row = (tid >> 3) + 32 * u;
    c.v[u] = *(const u32x4*)(base + (int64_t)min(r0 + row, T - 1) * rs + (tid & 7) * 8);
    if (r0 + row >= T) c.v[u] = u32x4{0u, 0u, 0u, 0u};
  }
}
__device__ inline void chunk_stash(const ChunkRegs& c, u32x4* s, int tid) {
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int row = (tid >> 3) + 32 * u;
    s[row * 8 + ((tid & 7) ^ swz(row))] = c.v[u];
  }
}

__global__ __launch_bounds__(256, 2) void attn_fwd_long_kernel(const bf16* __restrict__ qkv, int T, int H, int heads_total,
                                                            bf16* __restrict__ out, float* __restrict__ lse,
                                                            float* __restrict__ cls_prob) {
  __shared__ u32x4 Ks[LC * 8], Vs[LC * 8];
  __shared__ __attribute__((aligned(16))) float cls_s[LONG_T];
  static_assert(__alignof__(cls_s) >= 16, "written four keys at a time");
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lr = lane & 31, lh = lane >> 5;
  const int head = blockIdx.x % heads_total, b = head / H, h = head % H, D = H * HD;
  const int q0 = (blockIdx.x / heads_total) * 128 + wave * 32, qi = q0 + lr;
  const int64_t rs = 3 * (int64_t)D;
  const bf16* base = qkv + (int64_t)b * T * rs + h * HD;
  bf16x8 qf[4];
  const bf16* qrow = base + (int64_t)min(qi, T - 1) * rs;
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) qf[ks] = *(const bf16x8*)(qrow + (2 * ks + lh) * 8);
  const float c = 0.125f * 1.44269504088896341f;    // 1/sqrt(64) * log2(e)
  float m = -INFINITY, l = 0.f;                     // running maximum of the raw scores, running sum
  f32x16 o[2];
#pragma unroll
  for (int nb = 0; nb < 2; ++nb)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[nb][r] = 0.f;
  const bool cls_wave = cls_prob && q0 == 0;
  const int sw = swz(lr);
  ChunkRegs kr, vr;
  chunk_fetch(kr, base + D, rs, 0, T, tid);
  chunk_fetch(vr, base + 2 * D, rs, 0, T, tid);
  for (int c0 = 0; c0 < T; c0 += LC) {
    if (c0) __syncthreads();
    chunk_stash(kr, Ks, tid);
    chunk_stash(vr, Vs, tid);
    __syncthreads();
    if (c0 + LC < T) {
      chunk_fetch(kr, base + D, rs, c0 + LC, T, tid);
      chunk_fetch(vr, base + 2 * D, rs, c0 + LC, T, tid);
    }
    if (q0 >= T) continue;                            // (it only stages)
    f32x16 s[LCB];
    float mx = m;
#pragma unroll
    for (int jb = 0; jb < LCB; ++jb) {
      if (c0 + jb * 32 >= T) break;
#pragma unroll
      for (int r = 0; r < 16; ++r) s[jb][r] = 0.f;
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        const bf16x8 kf = *(const bf16x8*)(Ks + (jb * 32 + lr) * 8 + ((2 * ks + lh) ^ sw));
        s[jb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[ks], s[jb], 0, 0, 0);
      }
      if (c0 + jb * 32 + 32 > T) {
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (c0 + key_of(jb, r, lh) >= T) s[jb][r] = -INFINITY;
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[jb][r]);
    }
    if (cls_wave && lr == 0)
#pragma unroll
      for (int jb = 0; jb < LCB; ++jb) {
        if (c0 + jb * 32 >= T) break;
#pragma unroll
        for (int r = 0; r < 16; r += 4)
          *(float4*)(cls_s + c0 + key_of(jb, r, lh)) = make_float4(s[jb][r], s[jb][r + 1], s[jb][r + 2], s[jb][r + 3]);
      }
    mx = half_max(mx);         // finite: a chunk holds at least one key
    const float alpha = __builtin_amdgcn_exp2f((m - mx) * c), mc = mx * c;
    if (__any(mx != m)) {      // (else alpha is 1)
#pragma unroll
      for (int nb = 0; nb < 2; ++nb)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[nb][r] *= alpha;
    }
    m = mx;
    float sum = 0.f;
#pragma unroll
    for (int jb = 0; jb < LCB; ++jb) {
      if (c0 + jb * 32 >= T) break;
      Split p[2];
#pragma unroll
      for (int r = 0; r < 16; r += 2) {
        const float p0 = __builtin_amdgcn_exp2f(fmaf(s[jb][r], c, -mc)), p1 = __builtin_amdgcn_exp2f(fmaf(s[jb][r + 1], c, -mc));
        sum += p0;
        sum += p1;
        p[r >> 3].set2(r & 7, p0, p1);
      }
#pragma unroll
      for (int nb = 0; nb < 2; ++nb)
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) {
          const bf16x8 vf = lds_frag_t(Vs, nb, lane, 2 * jb + hf);
          o[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, p[hf].hi, o[nb], 0, 0, 0);
          o[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, p[hf].lo, o[nb], 0, 0, 0);
        }
    }
    l = l * alpha + sum + half_other(sum);
  }
  const float inv = 1.0f / l;
  if (qi < T) {
    if (lse && lh == 0) lse[((int64_t)b * H + h) * T + qi] = m * 0.125f + logf(l);
    bf16* orow = out + ((int64_t)b * T + qi) * D + h * HD + 4 * lh;
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
      for (int rq = 0; rq < 4; ++rq) {
        bf16x4 v4;
#pragma unroll
        for (int e = 0; e < 4; ++e) v4[e] = (bf16)(o[nb][4 * rq + e] * inv);
        *(bf16x4*)(orow + nb * 32 + 8 * rq) = v4;
      }
  }
  if (cls_prob && q0 - wave * 32 == 0) {            // the workgroup of the CLS query: its softmax row in fp32 (Eq. 6)
    __syncthreads();
    float* red = (float*)Ks;
    if (tid == 0) { red[0] = m; red[1] = inv; }
    __syncthreads();
    const float m0 = red[0] * c, i0 = red[1];
    for (int j = tid; j < T; j += 256) cls_prob[((int64_t)b * H + h) * T + j] = __builtin_amdgcn_exp2f(fmaf(cls_s[j], c, -m0)) * i0;
  }
}

// Backward beyond 256 tokens, two launches.  First delta_i = sum_j P_ij dP_ij in fp32, workgroups of 128 queries walking chunks of
// keys (dO . O would be one product, but of an output that has been rounded to bf16).  Then workgroups of the first half own
// 128 queries (dQ, chunks of keys), those of the second half 128 keys (dK and dV, chunks of queries).  (delta and dQ in one
// launch, dK and dV in another: 91 us at 577 tokens, 16 images of 6 heads, and 54 at 2 images; so 87 and 36.)
struct LongHead {                          // what a workgroup of these kernels works on
  const bf16 *base, *dobase;               // q of the head's first row (k, v: D and 2 D further), dO
  int64_t rs, row0;                        // elements from row to row of qkv; index of the head's first row in lse and delta
  int D, block;
  __device__ LongHead(const bf16* qkv, const bf16* dout, int T, int H, int heads_total) {
    const int head = blockIdx.x % heads_total, b = head / H, h = head % H;
    D = H * HD;
    rs = 3 * (int64_t)D;
    base = qkv + (int64_t)b * T * rs + h * HD;
    dobase = dout + (int64_t)b * T * D + h * HD;
    row0 = (int64_t)head * T;
    block = blockIdx.x / heads_total;
  }
};
// four 16-byte pieces of a row: the operand fragments of a wavefront's 32 rows
__device__ __forceinline__ void row_frags(bf16x8 (&f)[4], const bf16* row, int lh) {
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) f[ks] = *(const bf16x8*)(row + (2 * ks + lh) * 8);
}
// scores and dP of 32 staged rows (of xs and ys, from row r0 on) with the fragments xf and yf
__device__ __forceinline__ void score_products(f32x16& sa, f32x16& dp, const u32x4* xs, const u32x4* ys, int row, int lh, const bf16x8 (&xf)[4],
                                               const bf16x8 (&yf)[4]) {
#pragma unroll
  for (int r = 0; r < 16; ++r) { sa[r] = 0.f; dp[r] = 0.f; }
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) {
    sa = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lds_frag(xs, row, 2 * ks + lh), xf[ks], sa, 0, 0, 0);
    dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lds_frag(ys, row, 2 * ks + lh), yf[ks], dp, 0, 0, 0);
  }
}
constexpr float LOG2E = 1.44269504088896341f, SCORE2 = 0.125f * LOG2E;      // scores are divided by sqrt(64)
// P of a block of keys k0 .. k0 + 31 in place of the scores; 0 past the last key
__device__ __forceinline__ void block_probs(f32x16& sa, float l2, int k0, int lh, int T) {
#pragma unroll
  for (int r = 0; r < 16; ++r) sa[r] = __builtin_amdgcn_exp2f(sa[r] * SCORE2 - l2);
  if (k0 + 32 > T) {                       // uniform: this block reaches past the last key
#pragma unroll
    for (int r = 0; r < 16; ++r)
      if (k0 + key_of(0, r, lh) >= T) sa[r] = 0.f;
  }
}

__global__ __launch_bounds__(256, 2) void attn_delta_long_kernel(const bf16* __restrict__ qkv, const bf16* __restrict__ dout,
                                                                 const float* __restrict__ lse, int T, int H, int heads_total,
                                                                 float* __restrict__ delta) {
  __shared__ u32x4 Ks[LC * 8], Vs[LC * 8];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lr = lane & 31, lh = lane >> 5;
  const LongHead hd(qkv, dout, T, H, heads_total);
  const int q0 = hd.block * 128 + wave * 32, qi = q0 + lr, qc = min(qi, T - 1);
  bf16x8 qf[4], dof[4];
  row_frags(qf, hd.base + (int64_t)qc * hd.rs, lh);
  row_frags(dof, hd.dobase + (int64_t)qc * hd.D, lh);
  const float l2 = lse[hd.row0 + qc] * LOG2E;
  float dl = 0.f;
  ChunkRegs kr, vr;
  chunk_fetch(kr, hd.base + hd.D, hd.rs, 0, T, tid);
  chunk_fetch(vr, hd.base + 2 * hd.D, hd.rs, 0, T, tid);
  for (int c0 = 0; c0 < T; c0 += LC) {
    if (c0) __syncthreads();
    chunk_stash(kr, Ks, tid);
    chunk_stash(vr, Vs, tid);
    __syncthreads();
    if (c0 + LC < T) {
      chunk_fetch(kr, hd.base + hd.D, hd.rs, c0 + LC, T, tid);
      chunk_fetch(vr, hd.base + 2 * hd.D, hd.rs, c0 + LC, T, tid);
    }
    if (q0 >= T) continue;                            // (it only stages)
#pragma unroll
    for (int jb = 0; jb < LCB; ++jb) {
      if (c0 + jb * 32 >= T) break;
      f32x16 sa, dp;
      score_products(sa, dp, Ks, Vs, jb * 32 + lr, lh, qf, dof);
      block_probs(sa, l2, c0 + jb * 32, lh, T);
#pragma unroll
      for (int r = 0; r < 16; ++r) dl = fmaf(sa[r], dp[r], dl);
    }
  }
  dl = half_sum(dl);
  if (lh == 0 && qi < T) delta[hd.row0 + qi] = dl;
}

__global__ __launch_bounds__(256, 2) void attn_bwd_long_kernel(const bf16* __restrict__ qkv, const bf16* __restrict__ dout,
                                                               const float* __restrict__ lse, const float* __restrict__ delta, int T,
                                                               int H, int heads_total, bf16* __restrict__ dqkv) {
  __shared__ u32x4 As[LC * 8], Bs[LC * 8];
  __shared__ __attribute__((aligned(16))) float lse_s[LC], del_s[LC];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lr = lane & 31, lh = lane >> 5;
  const LongHead hd(qkv, dout, T, H, heads_total);
  const int nblk = (T + 127) / 128;
  bf16* dst = dqkv + (hd.base - qkv) + lr;           // feature lr of the head's first row of dq
  ChunkRegs ra, rb;
  if (hd.block < nblk) {
    const int q0 = hd.block * 128 + wave * 32, qc = min(q0 + lr, T - 1);
    bf16x8 qf[4], dof[4];
    row_frags(qf, hd.base + (int64_t)qc * hd.rs, lh);
    row_frags(dof, hd.dobase + (int64_t)qc * hd.D, lh);
    const float l2 = lse[hd.row0 + qc] * LOG2E, dl = delta[hd.row0 + qc];
    f32x16 o[2];
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[nb][r] = 0.f;
    chunk_fetch(ra, hd.base + hd.D, hd.rs, 0, T, tid);
    chunk_fetch(rb, hd.base + 2 * hd.D, hd.rs, 0, T, tid);
    for (int c0 = 0; c0 < T; c0 += LC) {
      if (c0) __syncthreads();
      chunk_stash(ra, As, tid);
      chunk_stash(rb, Bs, tid);
      __syncthreads();
      if (c0 + LC < T) {
        chunk_fetch(ra, hd.base + hd.D, hd.rs, c0 + LC, T, tid);
        chunk_fetch(rb, hd.base + 2 * hd.D, hd.rs, c0 + LC, T, tid);
      }
      if (q0 >= T) continue;
#pragma unroll
      for (int jb = 0; jb < LCB; ++jb) {
        if (c0 + jb * 32 >= T) break;
        f32x16 sa, dp;
        score_products(sa, dp, As, Bs, jb * 32 + lr, lh, qf, dof);
        block_probs(sa, l2, c0 + jb * 32, lh, T);
        Split ds[2];                                 // (the 1/8 of dS is applied to the sums)
#pragma unroll
        for (int r = 0; r < 16; r += 2) ds[r >> 3].set2(r & 7, sa[r] * (dp[r] - dl), sa[r + 1] * (dp[r + 1] - dl));
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
#pragma unroll
          for (int hf = 0; hf < 2; ++hf) {
            const bf16x8 kf = lds_frag_t(As, nb, lane, 2 * jb + hf);
            o[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ds[hf].hi, kf, o[nb], 0, 0, 0);
            o[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ds[hf].lo, kf, o[nb], 0, 0, 0);
          }
      }
    }
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int i = q0 + key_of(0, r, lh);
        if (i < T) dst[i * hd.rs + nb * 32] = (bf16)(o[nb][r] * 0.125f);
      }
    return;
  }
  const int j0 = (hd.block - nblk) * 128 + wave * 32, jc = min(j0 + lr, T - 1);
  bf16x8 kf[4], vf[4];
  row_frags(kf, hd.base + (int64_t)jc * hd.rs + hd.D, lh);
  row_frags(vf, hd.base + (int64_t)jc * hd.rs + 2 * hd.D, lh);
  f32x16 ok[2], ov[2];
#pragma unroll
  for (int nb = 0; nb < 2; ++nb)
#pragma unroll
    for (int r = 0; r < 16; ++r) { ok[nb][r] = 0.f; ov[nb][r] = 0.f; }
  chunk_fetch(ra, hd.base, hd.rs, 0, T, tid);
  chunk_fetch(rb, hd.dobase, hd.D, 0, T, tid);
  for (int c0 = 0; c0 < T; c0 += LC) {
    if (c0) __syncthreads();
    chunk_stash(ra, As, tid);
    chunk_stash(rb, Bs, tid);
    if (tid < LC) {
      lse_s[tid] = c0 + tid < T ? lse[hd.row0 + c0 + tid] * LOG2E : INFINITY;
      del_s[tid] = c0 + tid < T ? delta[hd.row0 + c0 + tid] : 0.f;
    }
    __syncthreads();
    if (c0 + LC < T) {
      chunk_fetch(ra, hd.base, hd.rs, c0 + LC, T, tid);
      chunk_fetch(rb, hd.dobase, hd.D, c0 + LC, T, tid);
    }
    if (j0 >= T) continue;
#pragma unroll
    for (int ib = 0; ib < LCB; ++ib) {
      if (c0 + ib * 32 >= T) break;
      f32x16 sa, dp;
      score_products(sa, dp, As, Bs, ib * 32 + lr, lh, kf, vf);
      Split p[2], ds[2];
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {              // queries c0 + 32 ib + 8 g4 + 4 lh + {0..3}
        const float4 l4 = *(const float4*)(lse_s + ib * 32 + 8 * g4 + 4 * lh);
        const float4 d4 = *(const float4*)(del_s + ib * 32 + 8 * g4 + 4 * lh);
        const float lv[4] = {l4.x, l4.y, l4.z, l4.w};
        const float dv[4] = {d4.x, d4.y, d4.z, d4.w};
#pragma unroll
        for (int e = 0; e < 4; e += 2) {
          const int r = g4 * 4 + e;
          const float p0 = __builtin_amdgcn_exp2f(sa[r] * SCORE2 - lv[e]), p1 = __builtin_amdgcn_exp2f(sa[r + 1] * SCORE2 - lv[e + 1]);
          p[r >> 3].set2(r & 7, p0, p1);
          ds[r >> 3].set2(r & 7, p0 * (dp[r] - dv[e]), p1 * (dp[r + 1] - dv[e + 1]));
        }
      }
#pragma unroll
      for (int nb = 0; nb < 2; ++nb)
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) {
          const bf16x8 gf = lds_frag_t(Bs, nb, lane, 2 * ib + hf), qf = lds_frag_t(As, nb, lane, 2 * ib + hf);
          ov[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(p[hf].hi, gf, ov[nb], 0, 0, 0);
          ov[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(p[hf].lo, gf, ov[nb], 0, 0, 0);
          ok[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ds[hf].hi, qf, ok[nb], 0, 0, 0);
          ok[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ds[hf].lo, qf, ok[nb], 0, 0, 0);
        }
    }
  }
#pragma unroll
  for (int nb = 0; nb < 2; ++nb)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int j = j0 + key_of(0, r, lh);
      if (j < T) {
        dst[j * hd.rs + hd.D + nb * 32] = (bf16)(ok[nb][r] * 0.125f);
        dst[j * hd.rs + 2 * hd.D + nb * 32] = (bf16)ov[nb][r];
      }
    }
}

void launch_bwd_long(const bf16* qkv, const bf16* dout, const float* lse, int B, int T, int H, float* delta, bf16* dqkv, hipStream_t s) {
  const int grid = B * H * ((T + 127) / 128);
  attn_delta_long_kernel<<<grid, 256, 0, s>>>(qkv, dout, lse, T, H, B * H, delta);
  attn_bwd_long_kernel<<<2 * grid, 256, 0, s>>>(qkv, dout, lse, delta, T, H, B * H, dqkv);
}

}  // namespace

bool attn_mfma_supported(int T, int d) { return d == HD && T >= 1 && T <= LONG_T; }

void attn_fwd_mfma(const void* qkv, int B, int T, int H, void* out, float* lse, float* cls_prob, hipStream_t s) {
  const bf16* q = (const bf16*)qkv;
  bf16* o = (bf16*)out;
  switch ((T + 31) / 32) {
    case 1: launch_fwd<1>(q, B, T, H, o, lse, cls_prob, s); break;
    case 2: launch_fwd<2>(q, B, T, H, o, lse, cls_prob, s); break;
    case 3: launch_fwd<3>(q, B, T, H, o, lse, cls_prob, s); break;
    case 4: launch_fwd<4>(q, B, T, H, o, lse, cls_prob, s); break;
    case 5: launch_fwd<5>(q, B, T, H, o, lse, cls_prob, s); break;
    case 6: launch_fwd<6>(q, B, T, H, o, lse, cls_prob, s); break;
    case 7: launch_fwd<7>(q, B, T, H, o, lse, cls_prob, s); break;
    case 8: launch_fwd<8>(q, B, T, H, o, lse, cls_prob, s); break;
    default: attn_fwd_long_kernel<<<B * H * ((T + 127) / 128), 256, 0, s>>>(q, T, H, B * H, o, lse, cls_prob); break;
  }
}

void attn_bwd_mfma(const void* qkv, const void* out, const void* dout, const float* lse, int B, int T, int H,
                   float* delta, void* dqkv, hipStream_t s) {
  const bf16* q = (const bf16*)qkv;
  const bf16* o = (const bf16*)out;
  const bf16* d = (const bf16*)dout;
  bf16* g = (bf16*)dqkv;
  switch ((T + 31) / 32) {
    case 1: launch_bwd_one<1>(q, o, d, lse, B, T, H, delta, g, s); break;
    case 2: launch_bwd_one<2>(q, o, d, lse, B, T, H, delta, g, s); break;
    case 3: launch_bwd_one<3>(q, o, d, lse, B, T, H, delta, g, s); break;
    case 4: launch_bwd_one<4>(q, o, d, lse, B, T, H, delta, g, s); break;
    case 5: launch_bwd_one<5>(q, o, d, lse, B, T, H, delta, g, s); break;
    case 6: launch_bwd_one<6>(q, o, d, lse, B, T, H, delta, g, s); break;
    case 7: launch_bwd_one<7>(q, o, d, lse, B, T, H, delta, g, s); break;
    case 8: launch_bwd<8>(q, o, d, lse, B, T, H, delta, g, s); break;
    default: launch_bwd_long(q, d, lse, B, T, H, delta, g, s); break;
  }
}

}  // namespace bsr
