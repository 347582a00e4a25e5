// bf16 MFMA GEMMs for gfx950 (CDNA4), the hot kernels of the BSR step.
//
// Two forms, both C = epilogue(sum_k A(m,k) B(k,n)) with fp32 accumulation in
// v_mfma_f32_32x32x16_bf16 tiles staged through LDS:
//   NT: A[M,K] and B^T[N,K] both have the contraction index contiguous.  Covers the forward linears
//       (activations x bf16 weight copy stored [out,in]) and the input gradients of Eq. 2
//       (dY x weight copy stored [in,out]).
//   TN: A^T[K,M] and B[K,N] both have the contraction index strided (rows are tokens).  Covers the
//       weight gradients of Eq. 4, dW = X^T dY, contraction over all tokens of the batch.
//
// Block tile BM x BN x 64 shared by WM x WN wavefronts, each owning a wave tile of 32x32 MFMA tiles.
// Tiles come straight from global memory into two to four stages of LDS (gemm_ntd_kernel: every wavefront
// loads; gemm_pair_kernel and gemm_tn_kernel: wavefronts of their own do); products whose k-tiles cannot be
// loaded that way wait in registers while the k-tile before feeds the matrix cores (gemm_nt_kernel), and
// products of few rows share k between wavefronts (gemm_nt_few_kernel).  Workgroups are renumbered so that each XCD (the hardware deals consecutive
// workgroup ids round-robin over 8 XCDs) works on a contiguous range of tiles and its L2 sees whole
// operand panels.
#include <algorithm>
#include <iterator>
#include <utility>

#include "bsr_internal.h"

namespace bsr {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));   // a 16-byte chunk in registers

constexpr int BK = 64;        // k-tile: 64 bf16 = 8 chunks of 16 bytes per row
constexpr int NXCD = 8;

// GELU(u) = u Phi(u) and its derivative Phi(u) + u phi(u) with the exact (erf) Phi.  erf comes from
// the rational-exponential form of Abramowitz & Stegun 7.1.26, |error| <= 1.5e-7 (below 1e-6 in
// fp32 arithmetic): far below the resolution of the bf16 values these epilogues write, at a fraction
// of the instructions of erff.  Its exp(-x^2) with x = u / sqrt(2) is the Gaussian that phi(u) needs
// as well.  Its coefficients are halved, so that it is Phi that comes out: exact, and one product of 22 less.
__device__ inline float phi_as(float u, float& gauss) {
  const float x = u * 0.70710678118654752f, ax = fabsf(x);
  const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f, ax, 1.0f));
  float p = fmaf(0.5f * 1.061405429f, t, 0.5f * -1.453152027f);
  p = fmaf(p, t, 0.5f * 1.421413741f);
  p = fmaf(p, t, 0.5f * -0.284496736f);
  p = fmaf(p, t, 0.5f * 0.254829592f);
  gauss = __expf(-ax * ax);
  return 0.5f + copysignf(fmaf(-p * t, gauss, 0.5f), x);
}
__device__ inline float gelu_f(float u) {
  float gauss;
  return u * phi_as(u, gauss);
}
__device__ inline float gelu_grad_f(float u) {
  float gauss;
  const float cdf = phi_as(u, gauss);
  return fmaf(u * 0.39894228040143268f, gauss, cdf);
}

template <int V> struct IC { static constexpr int value = V; };   // compile-time flag for generic lambdas
// f(IC<0>{}), ..., f(IC<N-1>{}): a loop whose index is a compile-time constant in the body
template <class F, int... I> __device__ __forceinline__ void sfor_impl(F&& f, std::integer_sequence<int, I...>) { (f(IC<I>{}), ...); }
template <int N, class F> __device__ __forceinline__ void sfor(F&& f) { sfor_impl(f, std::make_integer_sequence<int, N>{}); }

// LDS chunk swizzle: 16 consecutive rows reading the same logical 16-byte chunk hit 16 different
// (row parity, chunk position) pairs, i.e. all 64 banks once; 8 consecutive rows hit 8 positions.
__device__ inline int swz(int row) { return (row & 7) ^ ((row >> 3) & 1); }

// Logical tile id of this workgroup: XCD x owns the contiguous range [start(x), start(x+1)).
__device__ inline int xcd_remap(int pid, int nblocks) {
  const int base = nblocks / NXCD, rem = nblocks % NXCD;
  const int x = pid % NXCD, local = pid / NXCD;
  return x * base + min(x, rem) + local;
}

// Grouped form: row tiles count group after group (a group's last tile may be partial).  Row tile mt belongs to the group whose
// weights, bias and rows (from m0 on, up to g.M) g then describes; false: past the last group, nothing to do.
template <int BM>
__device__ __forceinline__ bool group_tile(GemmDesc& g, int mt, int& m0) {
  for (int e = 0; e < g.groups; ++e) {
    const int r0 = g.grp_off[e], r1 = g.grp_off[e + 1], n = (r1 - r0 + BM - 1) / BM;
    if (mt < n) {
      m0 = r0 + mt * BM;
      g.M = r1;
      g.B = (const bf16*)g.B + (int64_t)e * g.b_gs;
      if (g.bias) g.bias += (int64_t)e * g.bias_gs;
      return true;
    }
    mt -= n;
  }
  return false;
}

// Eight consecutive columns of output row m, accumulated in fp32: the statistics of a folded LayerNorm, bias,
// positional embedding (with the row remap of the patch embedding), GELU with its stored pre-activation or
// GELU', the residual, and the store (16 bytes of bf16, or 32 bytes of fp32).
// extra: what it would read of memory for them (the stored input of a GELU', the residual), read ahead.
struct Extra8 {
  bf16x8 u, r;
  __device__ __forceinline__ void fetch(const GemmDesc& g, int m, int col) {
    const int64_t row = g.remap_np > 0 ? (int64_t)m + m / g.remap_np + 1 : m;
    if (g.act == ACT_GELU_BWD) u = *(const bf16x8*)((const bf16*)g.aux + row * g.ldc + col);
    if (!g.out_f32 && g.res) r = *(const bf16x8*)((const bf16*)g.res + row * (g.ldr ? g.ldr : g.ldc) + col);
  }
};
__device__ __forceinline__ void finish8(const GemmDesc& g, float (&v)[8], int m, int col, const float (&bias)[8],
                                        const float (&cs)[8], const float2* st, const Extra8* extra = nullptr) {
  if (st) {
    const float2 ms = *st;
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = ms.y * fmaf(-ms.x, cs[j], v[j]);
  }
#pragma unroll
  for (int j = 0; j < 8; ++j) v[j] += bias[j];
  int64_t row = m;
  if (g.remap_np > 0) {
    row = (int64_t)m + m / g.remap_np + 1;
    const float* pr = g.pos + (int64_t)(m % g.remap_np + 1) * g.N + col;
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] += pr[j];
  }
  const int64_t off = row * g.ldc + col;
  if (g.act == ACT_GELU) {
    if (g.aux) {
      bf16x8 u;
#pragma unroll
      for (int j = 0; j < 8; ++j) u[j] = (bf16)v[j];
      *(bf16x8*)((bf16*)g.aux + off) = u;
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = gelu_f(v[j]);
  } else if (g.act == ACT_GELU_BWD) {
    const bf16x8 u = extra ? extra->u : *(const bf16x8*)((const bf16*)g.aux + off);
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] *= gelu_grad_f((float)u[j]);
  }
  if (g.out_f32) {
    float* c = (float*)g.C + off;
    *(float4*)c = make_float4(v[0], v[1], v[2], v[3]);
    *(float4*)(c + 4) = make_float4(v[4], v[5], v[6], v[7]);
  } else {
    if (g.res) {
      const bf16x8 rr = extra ? extra->r : *(const bf16x8*)((const bf16*)g.res + (g.ldr ? row * g.ldr + col : off));
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] += (float)rr[j];
    }
    bf16x8 o;
#pragma unroll
    for (int j = 0; j < 8; ++j) o[j] = (bf16)v[j];
    *(bf16x8*)((bf16*)g.C + off) = o;
  }
}

// Epilogue of one wave tile.  The fp32 accumulators (element r of a 32x32 tile sits at row
// 8*(r/4) + 4*(lane/32) + r%4, column lane%32) go through a per-wave LDS patch, 32 rows at a time,
// and come back row-major so that each lane owns 8 consecutive columns of one row: bias, GELU,
// GELU', positional embedding and residual are applied on 8-wide vectors and C is written with
// 16-byte stores (32 bytes for fp32 output).
template <int MI, int NI>
__device__ __forceinline__ void epilogue(const GemmDesc& g, f32x16 (&acc)[MI][NI], int row0, int col0, int lane,
                                float* patch, const float2* rowstat = nullptr) {
  constexpr int TN = NI * 32, LDP = TN + 4;     // +4 floats: rows start in different banks
  constexpr int CPR = TN / 8;                   // 8-column chunks per row
  constexpr int RPI = 64 / CPR;                 // rows handled per pass of the wave
  const int lc = lane & 31, lh = lane >> 5;
  const int my_chunk = lane % CPR, my_row = lane / CPR;
  const int col = col0 + my_chunk * 8;
  const bool col_ok = col < g.N;                // N is a multiple of 8 on this path
  float bias[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) bias[j] = (g.bias && col_ok) ? g.bias[col + j] : 0.f;
  // folded LayerNorm: rowstat holds (mean, 1/std) of the wave tile's rows of A, cs the column sums of W'
  float cs[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) cs[j] = (rowstat && col_ok) ? g.ln_colsum[col + j] : 0.f;
  // (row blocks and passes are loops, the accumulators of block mi picked by a switch: written out, this code was
  // most of the kernel, and a launch that follows another kernel fetches its code anew)
#pragma nounroll
  for (int mi = 0; mi < MI; ++mi) {
    sfor<MI>([&](auto I) __attribute__((always_inline)) {
      constexpr int i = decltype(I)::value;
      if (mi != i) return;
#pragma unroll
      for (int ni = 0; ni < NI; ++ni)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          patch[(8 * (r >> 2) + 4 * lh + (r & 3)) * LDP + ni * 32 + lc] = acc[i][ni][r];
    });
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma nounroll
    for (int pass = 0; pass < 32 / RPI; ++pass) {
      const int lr = pass * RPI + my_row;
      const int m = row0 + mi * 32 + lr;
      if (m >= g.M || !col_ok) continue;
      float v[8];
      const float4 p0 = *(const float4*)(patch + lr * LDP + my_chunk * 8);
      const float4 p1 = *(const float4*)(patch + lr * LDP + my_chunk * 8 + 4);
      v[0] = p0.x; v[1] = p0.y; v[2] = p0.z; v[3] = p0.w; v[4] = p1.x; v[5] = p1.y; v[6] = p1.z; v[7] = p1.w;
      finish8(g, v, m, col, bias, cs, rowstat ? rowstat + mi * 32 + lr : nullptr);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
}

// ------------------------------------------------------------------------------------------ NT
// LDS tile: rows of 8 chunks (16 B each), chunk kc of row r stored at position kc ^ swz(r).
// Software pipeline of one k-tile (4 MFMA steps of k = 16):
//   step 0,1: MFMAs on fragment set s while the fragments of the next step load into set s^1
//   step 2  : as above; the registers holding k-tile kt+1 go to the other LDS buffer and the global
//             loads of k-tile kt+1+PF are issued into the registers just freed
//   barrier ; step 3: MFMAs of the last fragments while the first fragments of k-tile kt+1 load.
// PF register stages hold the k-tiles kt+1 .. kt+PF on their way from global memory (k-tile j in stage
// j % PF): with PF = 1 a load has one k-tile of matrix work to land, which a small tile that is alone on
// its CU finishes long before an L2 or HBM access returns; such tiles run with PF = 3.
// Rows beyond M (or N) are clamped to the last valid row: they only feed accumulators that are
// never stored.  KTAIL zero-fills chunks beyond K (K % 64 != 0).
// (A folded 8-wave kernel whose tiles leave room for two workgroups per CU is held to the 128 registers that
// two workgroups need: the row sums would otherwise push the 192 x 128 shape to 132 and halve its occupancy.)
template <int BM, int BN, int WM, int WN, bool KTAIL, int PF = 1, bool LNF = false>
__global__ __launch_bounds__(WM * WN * 64, (LNF && PF == 1 && WM * WN == 8 && (BM + BN) * 256 <= 80 * 1024) ? 4 : 1)
void gemm_nt_kernel(GemmDesc g) {
  static_assert(!LNF || !KTAIL, "the folded LayerNorm reads whole rows of A in whole k-tiles");
  constexpr int NT = WM * WN * 64;
  constexpr int TM = BM / WM, TN = BN / WN, MI = TM / 32, NI = TN / 32;
  constexpr int ACH = (BM * 8 + NT - 1) / NT, BCH = (BN * 8 + NT - 1) / NT;   // 16-byte chunks per thread per tile
  constexpr bool AEVEN = (BM * 8) % NT == 0, BEVEN = (BN * 8) % NT == 0;      // else the last chunk is partial
  static_assert(MI >= 1 && NI >= 1 && TM % 32 == 0 && TN % 32 == 0, "wave tiles are made of 32x32 MFMA tiles");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  u32x4* As = (u32x4*)smem;                    // [2][BM*8]
  u32x4* Bs = As + 2 * BM * 8;                 // [2][BN*8]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WN, wn = wave % WN;
  const int ntn = (g.N + BN - 1) / BN;
  const int tile = xcd_remap(blockIdx.x, (int)gridDim.x);
  int m0 = (tile / ntn) * BM;
  const int n0 = (tile % ntn) * BN;
  if (g.grp_off && !group_tile<BM>(g, tile / ntn, m0)) return;
  const bf16* __restrict__ A = (const bf16*)g.A;
  const bf16* __restrict__ Bt = (const bf16*)g.B;

  // per-thread chunk coordinates are the same for every k-tile
  const bf16* pa[ACH];
  const bf16* pb[BCH];
  int sa[ACH], sb[BCH];
  const int kc8 = (tid & 7) * 8;               // NT is a multiple of 8: every chunk of a thread has the same kc
  // (threads past the end of an uneven tile repeat its last row: same data, same LDS slot)
#pragma unroll
  for (int i = 0; i < ACH; ++i) {
    const int row = AEVEN ? (tid + NT * i) >> 3 : min((tid + NT * i) >> 3, BM - 1);
    pa[i] = A + (int64_t)min(m0 + row, g.M - 1) * g.a_rs + kc8;
    sa[i] = row * 8 + ((tid & 7) ^ swz(row));
  }
#pragma unroll
  for (int i = 0; i < BCH; ++i) {
    const int row = BEVEN ? (tid + NT * i) >> 3 : min((tid + NT * i) >> 3, BN - 1);
    pb[i] = Bt + (int64_t)min(n0 + row, g.N - 1) * g.b_cs + kc8;
    sb[i] = row * 8 + ((tid & 7) ^ swz(row));
  }
  u32x4 ra[PF][ACH], rb[PF][BCH];        // the next PF k-tiles wait here while the current one is multiplied
  auto fetch = [&](auto ST, int k0) __attribute__((always_inline)) {
    constexpr int st = decltype(ST)::value;
    if (KTAIL) {
      const bool oob = k0 + kc8 >= g.K;
      const int kk = oob ? 0 : k0;
#pragma unroll
      for (int i = 0; i < ACH; ++i) {
        ra[st][i] = *(const u32x4*)(pa[i] + kk - (oob ? kc8 : 0));
        if (oob) ra[st][i] = u32x4{0u, 0u, 0u, 0u};
      }
#pragma unroll
      for (int i = 0; i < BCH; ++i) {
        rb[st][i] = *(const u32x4*)(pb[i] + kk - (oob ? kc8 : 0));
        if (oob) rb[st][i] = u32x4{0u, 0u, 0u, 0u};
      }
    } else {
#pragma unroll
      for (int i = 0; i < ACH; ++i) ra[st][i] = *(const u32x4*)(pa[i] + k0);
#pragma unroll
      for (int i = 0; i < BCH; ++i) rb[st][i] = *(const u32x4*)(pb[i] + k0);
    }
  };
  // Folded LayerNorm (LNF): the workgroup sees every element of its rows of A on the way to LDS, so it
  // takes their mean and variance itself: each thread adds up its chunks (always the same 8 of the 64
  // columns of a k-tile, k-tiles in ascending order; two bf16 per dot instruction), and the 8 threads of a
  // row are combined after the last k-tile.  The order does not depend on the tile shape.
  float rsum[LNF ? ACH : 1], rsq[LNF ? ACH : 1];
#pragma unroll
  for (int i = 0; i < (LNF ? ACH : 1); ++i) rsum[i] = rsq[i] = 0.f;
  auto stash = [&](auto ST, int buf) __attribute__((always_inline)) {
    constexpr int st = decltype(ST)::value;
#pragma unroll
    for (int i = 0; i < ACH; ++i) As[buf * BM * 8 + sa[i]] = ra[st][i];
#pragma unroll
    for (int i = 0; i < BCH; ++i) Bs[buf * BN * 8 + sb[i]] = rb[st][i];
    if constexpr (LNF) {
      const bf16x2 ones = __builtin_bit_cast(bf16x2, 0x3f803f80u);
#pragma unroll
      for (int i = 0; i < ACH; ++i)
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          // (the empty asm pins the word in a register of its own: without it the compiler folds the
          // extract-and-cast of all four words of a chunk onto word 0)
          unsigned word = ra[st][i][w];
          asm("" : "+v"(word));
          const bf16x2 pr = __builtin_bit_cast(bf16x2, word);
          rsum[i] = __builtin_amdgcn_fdot2_f32_bf16(pr, ones, rsum[i], false);
          rsq[i] = __builtin_amdgcn_fdot2_f32_bf16(pr, pr, rsq[i], false);
        }
    }
  };

  f32x16 acc[MI][NI];
#pragma unroll
  for (int mi = 0; mi < MI; ++mi)
#pragma unroll
    for (int ni = 0; ni < NI; ++ni)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[mi][ni][r] = 0.f;

  const int lr = lane & 31, lh = lane >> 5;
  int offa[MI], offb[NI];
#pragma unroll
  for (int mi = 0; mi < MI; ++mi) offa[mi] = (wm * TM + mi * 32 + lr) * 8;
#pragma unroll
  for (int ni = 0; ni < NI; ++ni) offb[ni] = (wn * TN + ni * 32 + lr) * 8;
  const int sw = swz(lr);

  bf16x8 fa[2][MI], fb[2][NI];
  auto load_frags = [&](int set, const u32x4* Ab, const u32x4* Bb, int ks) __attribute__((always_inline)) {
    const int kc = (ks * 2 + lh) ^ sw;
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) fa[set][mi] = *(const bf16x8*)(Ab + offa[mi] + kc);
#pragma unroll
    for (int ni = 0; ni < NI; ++ni) fb[set][ni] = *(const bf16x8*)(Bb + offb[ni] + kc);
  };
  auto mma = [&](int set) __attribute__((always_inline)) {
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
      for (int ni = 0; ni < NI; ++ni)
        acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[set][mi], fb[set][ni], acc[mi][ni], 0, 0, 0);
  };

  const int nk = (g.K + BK - 1) / BK;
  // prologue: k-tile 0 into LDS buffer 0, k-tiles 1 .. PF in flight in the register stages
  fetch(IC<0>{}, 0);
  stash(IC<0>{}, 0);
  auto pro = [&](auto J) __attribute__((always_inline)) {
    constexpr int j = decltype(J)::value;
    if (j <= PF && j < nk) fetch(IC<j % PF>{}, j * BK);
  };
  pro(IC<1>{}); pro(IC<2>{}); pro(IC<3>{}); pro(IC<4>{});
  static_assert(PF >= 1 && PF <= 4, "");
  __syncthreads();
  load_frags(0, As, Bs, 0);
  // One k-tile.  ST: the register stage of k-tile kt + 1.  do_stash: k-tile kt + 1 exists (stage -> other
  // LDS buffer, and its first fragments are loaded after the barrier); do_fetch: k-tile kt + 1 + PF exists.
  // The steady-state loop has both set and no branches, so that the compiler can interleave the whole body.
  auto ktile = [&](auto ST, auto STEADY, bool do_stash, bool do_fetch, int kt) __attribute__((always_inline)) {
    constexpr bool steady = decltype(STEADY)::value != 0;      // both flags known to be set: no branches
    const int buf = kt & 1;
    const u32x4* Ab = As + buf * BM * 8;
    const u32x4* Bb = Bs + buf * BN * 8;
    load_frags(1, Ab, Bb, 1);
    mma(0);
    load_frags(0, Ab, Bb, 2);
    mma(1);
    load_frags(1, Ab, Bb, 3);
    if (steady || do_stash) stash(ST, buf ^ 1);
    if (steady || do_fetch) fetch(ST, (kt + 1 + PF) * BK);
    mma(0);
    __syncthreads();
    if (steady || do_stash) load_frags(0, As + (buf ^ 1) * BM * 8, Bs + (buf ^ 1) * BN * 8, 0);
    mma(1);
  };
  // k-tile kt + j of a run that starts at a multiple of PF has k-tile kt + j + 1 in stage (j + 1) % PF
  auto steady_one = [&](auto J, int kt) __attribute__((always_inline)) {
    constexpr int j = decltype(J)::value;
    if (j < PF) ktile(IC<(j + 1) % PF>{}, IC<1>{}, true, true, kt + j);
  };
  auto tail_one = [&](auto J, int kt) __attribute__((always_inline)) {
    constexpr int j = decltype(J)::value;
    if (j < 2 * PF && kt + j < nk) ktile(IC<(j + 1) % PF>{}, IC<0>{}, kt + j + 1 < nk, kt + j + 1 + PF < nk, kt + j);
  };
  int kt = 0;
  for (; kt + 2 * PF < nk; kt += PF) {      // every k-tile of the group stashes and fetches
    steady_one(IC<0>{}, kt); steady_one(IC<1>{}, kt); steady_one(IC<2>{}, kt); steady_one(IC<3>{}, kt);
  }
  // at most 2 PF k-tiles are left
  tail_one(IC<0>{}, kt); tail_one(IC<1>{}, kt); tail_one(IC<2>{}, kt); tail_one(IC<3>{}, kt);
  tail_one(IC<4>{}, kt); tail_one(IC<5>{}, kt); tail_one(IC<6>{}, kt); tail_one(IC<7>{}, kt);
  __syncthreads();
  // the tile buffers are free now: reuse them as per-wave epilogue patches
  float* patch = (float*)smem + wave * (32 * (TN + 4));
  // folded LayerNorm: (mean, 1/std) of the tile's rows go behind the epilogue patches (inside the tile
  // buffers, which are free by now, whenever those are the larger of the two)
  constexpr size_t LDS_PATCH = (size_t)WM * WN * 32 * (TN + 4) * sizeof(float);
  float2* rowstat = (float2*)(smem + LDS_PATCH);
  if constexpr (LNF) {
#pragma unroll
    for (int i = 0; i < ACH; ++i) {
      float sm = rsum[i], sq = rsq[i];
      sm += __shfl_xor(sm, 1); sq += __shfl_xor(sq, 1);
      sm += __shfl_xor(sm, 2); sq += __shfl_xor(sq, 2);
      sm += __shfl_xor(sm, 4); sq += __shfl_xor(sq, 4);
      const float mean = sm / (float)g.K;
      const float var = fmaxf(sq / (float)g.K - mean * mean, 0.f);
      const int row = AEVEN ? (tid + NT * i) >> 3 : min((tid + NT * i) >> 3, BM - 1);
      if ((tid & 7) == 0) rowstat[row] = make_float2(mean, rsqrtf(var + g.ln_eps));
    }
    __syncthreads();
  }
  epilogue<MI, NI>(g, acc, m0 + wm * TM, n0 + wn * TN, lane, patch, LNF ? rowstat + wm * TM : nullptr);
}

template <int BM, int BN, int WM, int WN, int PF = 1>
void launch_nt(const GemmDesc& g, hipStream_t s) {
  static bool attr_set = false;
  constexpr size_t lds_tiles = (size_t)2 * (BM + BN) * BK * sizeof(bf16);
  constexpr size_t lds_patch = (size_t)WM * WN * 32 * (BN / WN + 4) * sizeof(float);   // epilogue patches
  constexpr size_t lds = lds_tiles > lds_patch ? lds_tiles : lds_patch;
  constexpr size_t lds_stat = lds_patch + BM * sizeof(float2);           // (mean, 1/std) of the tile's rows behind the patches
  constexpr size_t lds_lnf = lds > lds_stat ? lds : lds_stat;
  if (!attr_set) {
    (void)hipFuncSetAttribute((const void*)gemm_nt_kernel<BM, BN, WM, WN, false, PF>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    (void)hipFuncSetAttribute((const void*)gemm_nt_kernel<BM, BN, WM, WN, true, PF>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    (void)hipFuncSetAttribute((const void*)gemm_nt_kernel<BM, BN, WM, WN, false, PF, true>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_lnf);
    attr_set = true;
  }
  // grouped: every group may end in one partial row tile
  const int tiles = ((g.M + BM - 1) / BM + (g.grp_off ? g.groups : 0)) * ((g.N + BN - 1) / BN);
  if (g.ln_colsum) gemm_nt_kernel<BM, BN, WM, WN, false, PF, true><<<tiles, WM * WN * 64, lds_lnf, s>>>(g);
  else if (g.K % BK == 0) gemm_nt_kernel<BM, BN, WM, WN, false, PF><<<tiles, WM * WN * 64, lds, s>>>(g);
  else gemm_nt_kernel<BM, BN, WM, WN, true, PF><<<tiles, WM * WN * 64, lds, s>>>(g);
}

// ------------------------------------------------------------------------------------------ NT, operands straight into LDS
// The same product for K a multiple of 64, built around three facts measured on gfx950: LDS takes writes from
// registers at only 64 - 72 bytes per clock, a wavefront that is alone on its SIMD has nobody to hide its waits,
// and under matrix load the clock is set by power.  So (1) the operand tiles go from global memory straight into
// LDS with global_load_lds_dwordx4 (lane l of a wavefront writes 16 bytes at M0 + 16 l: one instruction fills 8 tile
// rows of 8 chunks, and the chunk swizzle of the LDS tile is applied to the global address a lane reads), which
// costs no registers and no LDS-write instructions; (2) NST stages of (BM + BN) x 64 and ONE barrier per k-tile:
// at the barrier every wavefront has finished reading k-tile kt and its own part of k-tile kt + 1 has landed
// (s_waitcnt vmcnt counts such a load when its data is in LDS), so behind the barrier k-tile kt + NST can go into
// the stage of k-tile kt; (3) the order of the k-loop is written out, every MFMA followed by at most one fragment
// read or a few loads, and pinned with scheduling barriers (the compiler's own order bunches the reads in front
// of the MFMAs and waits for them).  Large shapes have wave tiles of 64 x 64 and
// more (128 x 64 in the 256 x 256 shape): per MFMA a wavefront reads 0.75 - 1 KB of fragments instead of the 1.5 KB of a 64 x 32
// wave tile.  Shapes that leave a CU one workgroup of few tiles run eight wavefronts on small wave tiles and three stages:
// there two wavefronts a SIMD and k-tiles in flight count for more (6304 x 768 x 3072, 192 x 128: four wavefronts and two stages
// 42.4 us, eight and three 35.1; 4416 x 768 x 3072, 128 x 128: 34.6 and 27.0; the loads alone take 23 of those 27).
// The MFMA operands are swapped (weight rows first), so an accumulator holds the TRANSPOSED 32 x 32 output tile:
// a lane owns one output row and four runs of four consecutive columns.  That lets the epilogue round to bf16
// before the tile goes through LDS whenever nothing has to be added in fp32 afterwards (8-byte LDS writes of four
// bf16 instead of sixteen 4-byte writes per tile), and use 16-byte LDS writes otherwise.
template <int N> __device__ __forceinline__ void wait_vmcnt() {
  __builtin_amdgcn_s_waitcnt((N & 0xF) | ((N >> 4) << 14) | (0x7 << 4) | (0xF << 8));
}
__device__ __forceinline__ void wait_lgkmcnt0() { __builtin_amdgcn_s_waitcnt(0xF | (0x3 << 14) | (0x7 << 4)); }
#define BSR_SCHED_FENCE() __builtin_amdgcn_sched_barrier(0)
#define BSR_GLOBAL_PTR(p) ((const void __attribute__((address_space(1)))*)(p))
#define BSR_LDS_VOID(p) ((void __attribute__((address_space(3)))*)(p))

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

// Epilogue of one wave tile whose accumulators hold transposed output tiles: element r of acc[mi][ni] is output
// row mi*32 + lane%32, column ni*32 + 8*(r/4) + 4*(lane/32) + r%4.  32 rows at a time go through a per-wave LDS
// patch and come back with a lane owning 8 consecutive columns of a row (16-byte global stores).
// The code is kept short on purpose: a launch that follows another kernel fetches its code anew, and a version of
// this epilogue with every row block and pass written out (13 700 of the kernel's 14 400 instructions) cost a
// launch about 3 us.  So the row blocks are a loop (the accumulators of block mi are picked by a switch, which
// is all that has to be written out per block) and so are the passes: the finishing code exists once.
// What an epilogue has to do, as a compile-time constant of the kernel: plain products, residuals, the GELU and the GELU' have kernels of their
// own, in which none of the other forms' branches, registers and code are left (256 x 256 tiles: 7 - 11 KB each, 17 KB with all of them in one);
// EPI_ANY looks at the description (fp32 results, the positional embedding, a layer's joint backward launch).
enum Epi { EPI_ANY, EPI_BIAS, EPI_RES, EPI_GELU, EPI_GELU_BWD };
template <int NI> struct EpiLanes {
  static constexpr int TN = NI * 32;
  static constexpr int CPR = TN / 8, RPP = 64 / CPR;       // 8-column chunks per row, rows per pass of the wave
  static constexpr int NPASS = (32 + RPP - 1) / RPP;       // (with 12 chunks per row 60 lanes work and the last pass is partial)
};
// What an epilogue adds or multiplies, asked for when the last loads of k-tiles are out: the bias, and the first row block's residual or stored input of a
// GELU'.  Behind the k-loop they are one more trip to memory of every tile
// (steps of 32 images: DeiT-S 1250 -> 1234 us, ViT-B the same; asked for ahead of the first tiles instead, those land later: ViT-B 0.3 % longer).
// A slot is 16 bytes: with nothing but a bias to add (`direct`) the bias in the order of the accumulators (wave tiles 32 columns wide), else
// the bias of the lane's eight columns in two slots and a slot for every pass of a row block.
template <int MI, int NI, Epi E> struct EpiAhead {
  using L = EpiLanes<NI>;
  static constexpr bool EARLY = MI * NI <= 8;      // (the 320 x 256 shape would spill 27 registers: it asks behind the k-loop)
  static constexpr bool BIAS_EARLY = NI == 1;       // (as many slots either way)
  static constexpr int SLOTS = 2 + L::NPASS;
  f32x4 slot[SLOTS];
  const bf16* extra;
  int64_t lde;
  bool direct, on, bwd;              // only a bias to add; something to read ahead; and that it is for a GELU'
  template <class P> __device__ __forceinline__ void one(const GemmDesc& g, int row0, int col, int my_row, bool col_ok, P) {
    constexpr int p = P::value;
    const int m = row0 + p * L::RPP + my_row;
    if (p * L::RPP + my_row < 32 && m < g.M && col_ok) slot[2 + p] = *(const f32x4*)(extra + (int64_t)m * lde + col);
  }
  // bias of columns col0 + 32 (i / 4) + 8 (i % 4) + 4 lh ..
  __device__ static __forceinline__ f32x4 direct_bias(const GemmDesc& g, int col0, int lane, int i) {
    const int c = col0 + (i >> 2) * 32 + 8 * (i & 3) + 4 * (lane >> 5);
    return g.bias && c < g.N ? *(const f32x4*)(g.bias + c) : f32x4{0.f, 0.f, 0.f, 0.f};
  }
  __device__ __forceinline__ void fetch(const GemmDesc& g, int row0, int col0, int lane) {
    direct = E == EPI_ANY ? !g.out_f32 && !g.res && g.remap_np == 0 && g.act == ACT_NONE : E == EPI_BIAS;
    bwd = E == EPI_ANY ? g.act == ACT_GELU_BWD : E == EPI_GELU_BWD;
    on = E == EPI_ANY ? !direct && !g.out_f32 && g.remap_np == 0 && (bwd ? !g.res : g.act == ACT_NONE) : E == EPI_RES || E == EPI_GELU_BWD;
    if constexpr (E == EPI_GELU) {
      if constexpr (BIAS_EARLY)
#pragma unroll
        for (int i = 0; i < 4 * NI; ++i) slot[i] = direct_bias(g, col0, lane, i);
      return;
    }
    extra = bwd ? (const bf16*)g.aux : (const bf16*)g.res;
    lde = bwd || !g.ldr ? g.ldc : g.ldr;
    if (direct) {
      if constexpr (BIAS_EARLY)
#pragma unroll
        for (int i = 0; i < 4 * NI; ++i) slot[i] = direct_bias(g, col0, lane, i);
      return;
    }
    const int my_row = lane / L::CPR, col = col0 + lane % L::CPR * 8;
    const bool ok = col < g.N;
#pragma unroll
    for (int i = 0; i < 2; ++i) slot[i] = E != EPI_GELU_BWD && g.bias && ok ? *(const f32x4*)(g.bias + col + 4 * i) : f32x4{0.f, 0.f, 0.f, 0.f};
    if (on) sfor<L::NPASS>([&](auto P) __attribute__((always_inline)) { one(g, row0, col, my_row, ok && my_row < L::RPP, P); });
  }
};
template <int MI, int NI, Epi E>
__device__ __forceinline__ void epilogue_t(const GemmDesc& g, f32x16 (&acc)[MI][NI], int row0, int col0, int lane,
                                           unsigned char* patch, EpiAhead<MI, NI, E>& early) {
  using L = EpiLanes<NI>;
  constexpr int TN = L::TN, CPR = L::CPR, RPP = L::RPP, NPASS = L::NPASS;
  const int lm = lane & 31, lh = lane >> 5;
  const int my_chunk = lane % CPR, my_row = lane / CPR;
  const int col = col0 + my_chunk * 8;
  const bool col_ok = col < g.N && my_row < RPP;    // N is a multiple of 8 on this path
  // nothing but the bias to add, or the GELU behind it: finished where the accumulators are, rounded first, so that half the bytes move.
  // The GELU is bound by the vector unit, two wavefronts a SIMD: on all values of a row block here it is one run of independent instructions; on eight
  // values a pass behind an fp32 patch, as it was, every pass waited for the patch and went through the forms' branches.  With a GELU, chains of
  // launches: 6304 x 3072 x 768 43.3 -> 39.3 us, 25216 rows 159 -> 154, 9232 x 1536 x 384 26.7 -> 22.7 (plain products 32.3 -> 32.0, 122 -> 121, 17.2 -> 17.1).
  if (E == EPI_GELU || early.direct) {
    constexpr int LDB = TN * 2 + 16;                // bytes per patch row
    using Ahead = EpiAhead<MI, NI, E>;
    f32x4 bq[4 * NI];                               // bias of the columns this lane holds
    auto read_bias = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < 4 * NI; ++i) bq[i] = Ahead::direct_bias(g, col0, lane, i);
    };
    if constexpr (Ahead::BIAS_EARLY)
#pragma unroll
      for (int i = 0; i < 4 * NI; ++i) bq[i] = early.slot[i];
    else if constexpr (Ahead::EARLY) read_bias();
    // a row block of NI accumulators rounded into the patch, and from there to dst: all rows of the lane on their way at once
    auto to_patch = [&](auto value) __attribute__((always_inline)) {
#pragma unroll
      for (int ni = 0; ni < NI; ++ni)
#pragma unroll
        for (int rg = 0; rg < 4; ++rg) {
          bf16x4 o;
#pragma unroll
          for (int e = 0; e < 4; ++e) o[e] = (bf16)value(ni, rg, e);
          *(bf16x4*)(patch + lm * LDB + (ni * 32 + 8 * rg + 4 * lh) * 2) = o;
        }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
    };
    const bool whole_cols = RPP * NPASS == 32 && RPP * CPR == 64 && col0 + TN <= g.N;
    auto out = [&](bf16* dst, int mi) __attribute__((always_inline)) {
      const int first = row0 + mi * 32, m = first + my_row;
      bf16* to = dst + (int64_t)m * g.ldc + col;
      if (whole_cols && first + 32 <= g.M) {        // (a whole row block: its stores behind each other, without a branch around each)
        bf16x8 row[NPASS];
#pragma unroll
        for (int p = 0; p < NPASS; ++p) row[p] = *(const bf16x8*)(patch + (p * RPP + my_row) * LDB + my_chunk * 16);
#pragma unroll
        for (int p = 0; p < NPASS; ++p) *(bf16x8*)(to + (int64_t)(p * RPP) * g.ldc) = row[p];
      } else {
#pragma nounroll
        for (int p = 0; p < NPASS; ++p)
          if (p * RPP + my_row < 32 && m + p * RPP < g.M && col_ok)
            *(bf16x8*)(to + (int64_t)(p * RPP) * g.ldc) = *(const bf16x8*)(patch + (p * RPP + my_row) * LDB + my_chunk * 16);
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
    };
#pragma nounroll
    for (int mi = 0; mi < MI; ++mi) {
      if constexpr (!Ahead::BIAS_EARLY && !Ahead::EARLY) read_bias();     // (once per row block: no registers to keep it in)
      if constexpr (E == EPI_GELU) {
        f32x16 blk[NI];                             // (the code of a row block's GELU exists once)
        sfor<MI>([&](auto I) __attribute__((always_inline)) {
          constexpr int i = decltype(I)::value;
          if (mi == i)
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) blk[ni] = acc[i][ni];
        });
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
#pragma unroll
          for (int r = 0; r < 16; ++r) blk[ni][r] += bq[4 * ni + r / 4][r % 4];
        if (g.aux) {                                // (its rows leave while the GELU is computed)
          to_patch([&](int ni, int rg, int e) __attribute__((always_inline)) { return blk[ni][4 * rg + e]; });
          out((bf16*)g.aux, mi);
        }
        to_patch([&](int ni, int rg, int e) __attribute__((always_inline)) { return gelu_f(blk[ni][4 * rg + e]); });
      } else {
        sfor<MI>([&](auto I) __attribute__((always_inline)) {
          constexpr int i = decltype(I)::value;
          if (mi == i) to_patch([&](int ni, int rg, int e) __attribute__((always_inline)) { return acc[i][ni][4 * rg + e] + bq[4 * ni + rg][e]; });
        });
      }
      out((bf16*)g.C, mi);
    }
    return;
  }
  constexpr int LDF = TN * 4 + 16;
  float bias[8], cs[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) { bias[j] = early.slot[j / 4][j % 4]; cs[j] = 0.f; }
  // A residual or the stored input of a GELU' is read NPASS passes ahead (the passes written out for it): read where it is
  // used, every pass of a wavefront waits for memory, 8 - 20 times a tile: 6304 x 768 x 768 19.1 -> 16.2 us (192 x 128),
  // 25216 x 768 x 768 41.9 -> 36.7 (320 x 256), launches in a row.
  const bool bwd = early.bwd;
#pragma nounroll
  for (int mi = 0; mi < MI; ++mi) {
    sfor<MI>([&](auto I) __attribute__((always_inline)) {
      constexpr int i = decltype(I)::value;
      if (mi != i) return;
#pragma unroll
      for (int ni = 0; ni < NI; ++ni)
#pragma unroll
        for (int rg = 0; rg < 4; ++rg)
          *(f32x4*)(patch + lm * LDF + (ni * 32 + 8 * rg + 4 * lh) * 4) =
              f32x4{acc[i][ni][4 * rg], acc[i][ni][4 * rg + 1], acc[i][ni][4 * rg + 2], acc[i][ni][4 * rg + 3]};
    });
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (early.on) {
      sfor<NPASS>([&](auto P) __attribute__((always_inline)) {
        constexpr int p = decltype(P)::value;
        const int lr = p * RPP + my_row;
        const int m = row0 + mi * 32 + lr;
        const bool mine = lr < 32 && m < g.M && col_ok;
        const bf16x8 e = __builtin_bit_cast(bf16x8, early.slot[2 + p]);
        if (mi + 1 < MI) early.one(g, row0 + (mi + 1) * 32, col, my_row, col_ok, P);
        if (mine) {
          const f32x4 p0 = *(const f32x4*)(patch + lr * LDF + my_chunk * 32);
          const f32x4 p1 = *(const f32x4*)(patch + lr * LDF + my_chunk * 32 + 16);
          const float v[8] = {p0[0], p0[1], p0[2], p0[3], p1[0], p1[1], p1[2], p1[3]};
          bf16x8 o;
          if (E == EPI_GELU_BWD) {
#pragma unroll
            for (int j = 0; j < 8; ++j) o[j] = (bf16)(v[j] * gelu_grad_f((float)e[j]));
          } else if (bwd) {
#pragma unroll
            for (int j = 0; j < 8; ++j) o[j] = (bf16)((v[j] + bias[j]) * gelu_grad_f((float)e[j]));
          } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) o[j] = (bf16)((v[j] + bias[j]) + (float)e[j]);
          }
          *(bf16x8*)((bf16*)g.C + (int64_t)m * g.ldc + col) = o;
        }
      });
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      continue;
    }
#pragma nounroll
    for (int p = 0; p < NPASS; ++p) {
      const int lr = p * RPP + my_row;
      const int m = row0 + mi * 32 + lr;
      if (lr >= 32 || m >= g.M || !col_ok) continue;
      const f32x4 p0 = *(const f32x4*)(patch + lr * LDF + my_chunk * 32);
      const f32x4 p1 = *(const f32x4*)(patch + lr * LDF + my_chunk * 32 + 16);
      float v[8] = {p0[0], p0[1], p0[2], p0[3], p1[0], p1[1], p1[2], p1[3]};
      finish8(g, v, m, col, bias, cs, nullptr);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
}

// The same for results that leave as plain fp32, as weight gradients do.  (Through epilogue_t, whose other paths the compiler cannot
// rule out, the kernels with the 256 x 128 weight-gradient tile spilled 25 - 29 registers and were 5 KB longer.)
template <int MI, int NI>
__device__ __forceinline__ void epilogue_f32(float* c, int64_t ldc, int M, int N, const f32x16 (&acc)[MI][NI], int row0, int col0, int lane,
                                             unsigned char* patch) {
  constexpr int TN = NI * 32, LDF = TN * 4 + 16, CPR = TN / 4, RPP = 64 / CPR;     // 4-column chunks per row, rows per pass of the wave
  static_assert(32 % RPP == 0, "whole passes");
  const int lm = lane & 31, lh = lane >> 5, my_chunk = lane % CPR, my_row = lane / CPR, col = col0 + my_chunk * 4;
#pragma nounroll
  for (int mi = 0; mi < MI; ++mi) {
    sfor<MI>([&](auto I) __attribute__((always_inline)) {
      constexpr int i = decltype(I)::value;
      if (mi != i) return;
#pragma unroll
      for (int ni = 0; ni < NI; ++ni)
#pragma unroll
        for (int rg = 0; rg < 4; ++rg)
          *(f32x4*)(patch + lm * LDF + (ni * 32 + 8 * rg + 4 * lh) * 4) =
              f32x4{acc[i][ni][4 * rg], acc[i][ni][4 * rg + 1], acc[i][ni][4 * rg + 2], acc[i][ni][4 * rg + 3]};
    });
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll 4
    for (int p = 0; p < 32 / RPP; ++p) {
      const int lr = p * RPP + my_row, m = row0 + mi * 32 + lr;
      if (m < M && col < N) *(f32x4*)(c + (int64_t)m * ldc + col) = *(const f32x4*)(patch + lr * LDF + my_chunk * 16);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
}

// The work of one tile (a kernel of its own below, and the input-gradient half of a layer's backward launch).
template <int BM, int BN, int WM, int WN, int NST, Epi E = EPI_ANY>
__device__ __forceinline__ void ntd_body(GemmDesc g, int tile) {
  constexpr int NT = WM * WN * 64;
  constexpr int TM = BM / WM, TN = BN / WN, MI = TM / 32, NI = TN / 32, NMF = MI * NI, NFR = MI + NI;
  constexpr int RPI = NT / 8;                       // tile rows one load instruction of the workgroup fills
  constexpr int AL = BM / RPI, BL = BN / RPI;       // load instructions per thread and k-tile
  constexpr int LPT = AL + BL;
  constexpr int STAGE = (BM + BN) * 128;            // bytes of a stage: rows of 8 chunks of 16 bytes, A rows first
  static_assert(BM % RPI == 0 && BN % RPI == 0 && RPI % 16 == 0, "a load instruction covers whole groups of 16 rows");
  static_assert(NST >= 2 && NST <= 4 && (NST - 1) * LPT <= 60, "vmcnt has 6 bits");
  static_assert(NMF >= 2 && NMF <= 16, "");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int ntn = (g.N + BN - 1) / BN;
  int m0 = (tile / ntn) * BM;
  const int n0 = (tile % ntn) * BN;
  if (g.grp_off && !group_tile<BM>(g, tile / ntn, m0)) return;
  const bf16* __restrict__ A = (const bf16*)g.A;
  const bf16* __restrict__ Bt = (const bf16*)g.B;

  // loader: thread t of load instruction i brings chunk kc of tile row i*RPI + t/8 to LDS slot (row, t%8); rows
  // past M (or N) repeat the last valid row: they only feed accumulators that are never stored
  const int lrow = tid >> 3;
  const int kc = (tid & 7) ^ swz(lrow);
  unsigned off[LPT];
#pragma unroll
  for (int i = 0; i < AL; ++i) off[i] = (unsigned)min(m0 + i * RPI + lrow, g.M - 1) * (unsigned)g.a_rs + kc * 8;
#pragma unroll
  for (int i = 0; i < BL; ++i) off[AL + i] = (unsigned)min(n0 + i * RPI + lrow, g.N - 1) * (unsigned)g.b_cs + kc * 8;
  auto issue1 = [&](auto I, int kt, int st) __attribute__((always_inline)) {
    constexpr int i = decltype(I)::value;
    const bf16* src = (i < AL ? A : Bt) + (size_t)kt * 64;
    unsigned char* dst = smem + st * STAGE + wave * 1024 + (i < AL ? i * RPI * 128 : BM * 128 + (i - AL) * RPI * 128);
    __builtin_amdgcn_global_load_lds(BSR_GLOBAL_PTR(src + off[i]), BSR_LDS_VOID(dst), 16, 0, 0);
  };

  f32x16 acc[MI][NI];
#pragma unroll
  for (int mi = 0; mi < MI; ++mi)
#pragma unroll
    for (int ni = 0; ni < NI; ++ni)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[mi][ni][r] = 0.f;

  // fragments: read order A0, B0 .. B(NI-1), A1 .. A(MI-1), so that the first MFMAs of a k-step can start early
  const int lr = lane & 31, lh = lane >> 5, sw = swz(lr);
  int offr[NFR];
  bf16x8 fr[2][NFR];
#pragma unroll
  for (int j = 0; j < NFR; ++j) {
    const bool isA = j == 0 || j > NI;
    const int idx = j == 0 ? 0 : (j <= NI ? j - 1 : j - NI);
    offr[j] = isA ? (wm * TM + idx * 32 + lr) * 128 : BM * 128 + (wn * TN + idx * 32 + lr) * 128;
  }
  auto rd1 = [&](auto SET, auto J, int st, int ks) __attribute__((always_inline)) {
    constexpr int set = decltype(SET)::value, j = decltype(J)::value;
    fr[set][j] = *(const bf16x8*)(smem + st * STAGE + (((ks * 2 + lh) ^ sw) << 4) + offr[j]);
  };
  auto mf1 = [&](auto SET, auto J) __attribute__((always_inline)) {
    constexpr int set = decltype(SET)::value, j = decltype(J)::value, mi = j / NI, ni = j % NI;
    constexpr int ja = mi == 0 ? 0 : NI + mi, jb = 1 + ni;
    acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[set][jb], fr[set][ja], acc[mi][ni], 0, 0, 0);
  };
  // The loads of a k-tile are spread evenly over the SPAN MFMAs behind the barrier that frees its stage.  A wavefront that issues loads faster than the CU's
  // path from L2 takes them (48 bytes per clock) stands still, and its MFMAs with it; issued later they land later.  So large wave tiles spread
  // them (all of a k-tile with three stages, half with two), small ones, whose k-tiles are short, issue them at once.  Chains of launches, at once -> spread:
  // 6304 x 768 x 3072 in 256 x 256 tiles 62.4 -> 58.8 us, in 320 x 256 75.2 -> 70.3, in 256 x 128 39.6 -> 36.3; 25216 x 768 x 3072 in 320 x 256 110.4 -> 107.5;
  // 192 x 256 and 256 x 192 tiles 1.01 .. 1.08 as long, 128 x 128 and 128 x 64 tiles of 132 workgroups (in a step) 1.02 and 1.04.
  constexpr int PRE = NMF >= 16 ? 4 : (NMF >= 8 ? 2 : 1);         // MFMAs of the last k-step in front of the barrier
  constexpr int POST = NMF - PRE;
  constexpr int SPAN = POST + (NST == 2 ? NMF >= 8 : NMF >= 4 ? 3 : NMF == 3 ? 2 : 0) * NMF;    // MFMAs that the loads of a k-tile are spread over
  auto loads_at = [&](auto P, int kt, int st) __attribute__((always_inline)) {
    constexpr int p = decltype(P)::value, lo = p >= SPAN ? LPT : (p * LPT + SPAN - 1) / SPAN, hi = p + 1 >= SPAN ? LPT : ((p + 1) * LPT + SPAN - 1) / SPAN;
    sfor<hi - lo>([&](auto L) __attribute__((always_inline)) { issue1(IC<lo + decltype(L)::value>{}, kt, st); });
  };
  constexpr bool LATE = SPAN > POST;                              // some follow in the next k-tile
  // one k-step: MFMAs on fragment set SET; the fragments of (stage st, k-step ks) go into the other set; LOADS: with its share of the loads of
  // k-tile ktl into stage stl
  auto kstep = [&](auto SET, auto LOADS, auto KS, int st, int ktl, int stl) __attribute__((always_inline)) {
    constexpr int set = decltype(SET)::value, ks = decltype(KS)::value;
    sfor<NMF>([&](auto J) __attribute__((always_inline)) {
      constexpr int j = decltype(J)::value;
      mf1(IC<set>{}, J);
      constexpr int RPM = (NFR + NMF - 1) / NMF;         // reads behind an MFMA
      sfor<RPM>([&](auto R) __attribute__((always_inline)) {
        constexpr int r = j * RPM + decltype(R)::value;
        if constexpr (r < NFR) rd1(IC<set ^ 1>{}, IC<r>{}, st, ks);
      });
      if constexpr (decltype(LOADS)::value) loads_at(IC<POST + (ks - 1) * NMF + j>{}, ktl, stl);
      BSR_SCHED_FENCE();
    });
  };
  // The last k-step of k-tile kt (fragments in set 1) with the barrier.  VMW >= 0: loads that may stay in flight
  // at the barrier (steady state, the first loads of k-tile kt + NST follow it); VMW < 0: tail, nothing is issued and the
  // count follows from rem, the number of k-tiles after this one (after the last one barrier and reads are idle).
  auto klast = [&](auto VMW, int kt, int st, int stn, int rem) __attribute__((always_inline)) {
    constexpr int vmw = decltype(VMW)::value;
    constexpr int RPP = (NFR + POST - 1) / POST;
    sfor<PRE>([&](auto J) __attribute__((always_inline)) { mf1(IC<1>{}, J); BSR_SCHED_FENCE(); });
    wait_lgkmcnt0();
    if constexpr (vmw >= 0) wait_vmcnt<vmw>();
    else if (rem >= 3) wait_vmcnt<2 * LPT>();
    else if (rem == 2) wait_vmcnt<LPT>();
    else wait_vmcnt<0>();
    __builtin_amdgcn_s_barrier();
    BSR_SCHED_FENCE();
    sfor<POST>([&](auto P) __attribute__((always_inline)) {
      constexpr int p = decltype(P)::value;
      mf1(IC<1>{}, IC<PRE + p>{});
      sfor<RPP>([&](auto R) __attribute__((always_inline)) {
        constexpr int r = p * RPP + decltype(R)::value;
        if constexpr (r < NFR) rd1(IC<0>{}, IC<r>{}, stn, 0);
      });
      if constexpr (vmw >= 0) loads_at(P, kt + NST, st);
      BSR_SCHED_FENCE();
    });
  };

  const int nk = g.K / BK;
  EpiAhead<MI, NI, E> early;
  // prologue: every stage filled (k-tiles 0 .. NST-1), k-tile 0 landed
#pragma unroll
  for (int j = 0; j < NST; ++j)
    if (j < nk) sfor<LPT>([&](auto I) __attribute__((always_inline)) { issue1(I, j, j); });
  {
    const int fl = min(nk, NST) - 1;            // k-tiles that may stay in flight
    if (fl >= 3) wait_vmcnt<3 * LPT>(); else if (fl == 2) wait_vmcnt<2 * LPT>(); else if (fl == 1) wait_vmcnt<LPT>(); else wait_vmcnt<0>();
  }
  __builtin_amdgcn_s_barrier();
  sfor<NFR>([&](auto J) __attribute__((always_inline)) { rd1(IC<0>{}, J, 0, 0); });
  int st = 0, kt = 0;
  // a k-tile; LOADS: with the late loads of k-tile kt + NST - 1, whose stage the barrier before this one freed
  auto ktile = [&](auto LOADS, auto VMW) __attribute__((always_inline)) {
    const int stn = (st + 1 == NST) ? 0 : st + 1, stl = st == 0 ? NST - 1 : st - 1;
    kstep(IC<0>{}, LOADS, IC<1>{}, st, kt + NST - 1, stl);
    kstep(IC<1>{}, LOADS, IC<2>{}, st, kt + NST - 1, stl);
    kstep(IC<0>{}, LOADS, IC<3>{}, st, kt + NST - 1, stl);
    klast(VMW, kt, st, stn, nk - 1 - kt);
    st = stn;
    ++kt;
  };
  constexpr IC<(NST - 2) * LPT> steady{};
  if constexpr (LATE) {
    if (kt + NST < nk) ktile(IC<0>{}, steady);                    // (the prologue's loads are all out)
    while (kt + NST < nk) ktile(IC<1>{}, steady);
    if (kt > 0) ktile(IC<1>{}, IC<-1>{});                         // the last late loads
  } else {
    while (kt + NST < nk) ktile(IC<0>{}, steady);
  }
  if constexpr (early.EARLY) early.fetch(g, m0 + wm * TM, n0 + wn * TN, lane);
  while (kt < nk) ktile(IC<0>{}, IC<-1>{});                       // nothing left to issue
  if constexpr (!early.EARLY) early.fetch(g, m0 + wm * TM, n0 + wn * TN, lane);
  // every wavefront is past the last barrier, i.e. has read its last fragments: the stages are free
  epilogue_t<MI, NI, E>(g, acc, m0 + wm * TM, n0 + wn * TN, lane, smem + wave * (32 * (TN * 4 + 16)), early);
}

// What a product's first loads need, as plain kernel arguments in front: the first 14 dwords come in registers with the wavefront
// (-amdgpu-kernarg-preload-count), a description passed by value is a trip to memory first.  The present kernels without and
// with it: one image through the ViT-B encoder (65 launches) 431 -> 410 us, steps of 32 images DeiT-S 1201 -> 1170, ViT-B 2216 -> 2192.
#define BSR_HOT_PARAMS const void *hA, const void *hB, int hM, int hN, int hK, unsigned ha_rs, unsigned hb_cs, int tiles
#define BSR_HOT_ARGS(g, tiles) (g).A, (g).B, (g).M, (g).N, (g).K, (unsigned)(g).a_rs, (unsigned)(g).b_cs, tiles
#define BSR_HOT_INTO(g) ((g).A = hA, (g).B = hB, (g).M = hM, (g).N = hN, (g).K = hK, (g).a_rs = ha_rs, (g).b_cs = hb_cs)

// (a shape whose stages take at most half of the 160 KB is held to the registers that let two workgroups share a CU)
template <int BM, int BN, int WM, int WN, int NST, Epi E>
__global__ __launch_bounds__(WM * WN * 64, NST * (BM + BN) * 128 <= 80 * 1024 ? WM * WN / 2 : 1)
void gemm_ntd_kernel(BSR_HOT_PARAMS, const int32_t* grp_off, GemmDesc g) {
  BSR_HOT_INTO(g);
  g.grp_off = grp_off;
  ntd_body<BM, BN, WM, WN, NST, E>(g, xcd_remap(blockIdx.x, tiles));
}

Epi epi_of(const GemmDesc& g) {
  if (g.out_f32 || g.remap_np > 0) return EPI_ANY;
  if (g.act == ACT_NONE) return g.res ? EPI_RES : EPI_BIAS;
  if (g.res) return EPI_ANY;
  return g.act == ACT_GELU ? EPI_GELU : g.act == ACT_GELU_BWD && !g.bias ? EPI_GELU_BWD : EPI_ANY;
}

template <int BM, int BN, int WM, int WN, int NST, Epi E>
void launch_ntd_as(const GemmDesc& g, hipStream_t s) {
  static bool attr_set = false;
  constexpr size_t lds_tiles = (size_t)NST * (BM + BN) * 128;
  constexpr size_t lds_patch = (size_t)WM * WN * 32 * ((BN / WN) * 4 + 16);
  static_assert(lds_patch <= lds_tiles, "the epilogue patches live in the stage buffers");
  auto kern = gemm_ntd_kernel<BM, BN, WM, WN, NST, E>;
  if (!attr_set) {
    (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_tiles);
    attr_set = true;
  }
  // grouped: every group may end in one partial row tile
  const int tiles = ((g.M + BM - 1) / BM + (g.grp_off ? g.groups : 0)) * ((g.N + BN - 1) / BN);
  kern<<<tiles, WM * WN * 64, lds_tiles, s>>>(BSR_HOT_ARGS(g, tiles), g.grp_off, g);
}
template <int BM, int BN, int WM, int WN, int NST>
void launch_ntd(const GemmDesc& g, hipStream_t s) {
  switch (epi_of(g)) {
    case EPI_BIAS: launch_ntd_as<BM, BN, WM, WN, NST, EPI_BIAS>(g, s); break;
    case EPI_RES: launch_ntd_as<BM, BN, WM, WN, NST, EPI_RES>(g, s); break;
    case EPI_GELU: launch_ntd_as<BM, BN, WM, WN, NST, EPI_GELU>(g, s); break;
    case EPI_GELU_BWD: launch_ntd_as<BM, BN, WM, WN, NST, EPI_GELU_BWD>(g, s); break;
    default: launch_ntd_as<BM, BN, WM, WN, NST, EPI_ANY>(g, s); break;
  }
}
// The kernels that load straight into LDS hold an operand's row offsets in 32 bits (elements): larger operands, such as the
// activations of 8192 images, go to the register-staged kernels, whose offsets have 64.
bool offsets_fit(const GemmDesc& g) {
  return (int64_t)g.M * g.a_rs <= (int64_t)UINT32_MAX && (int64_t)g.N * g.b_cs <= (int64_t)UINT32_MAX;
}
// what the direct-to-LDS kernels take: whole k-tiles, no folded LayerNorm
bool is_ntd(const GemmDesc& g) { return g.K % BK == 0 && !g.ln_colsum && offsets_fit(g); }

// ------------------------------------------------------------------------------------------ NT, few rows
// The same product where block tiles shared by eight wavefronts would leave most CUs idle.  A workgroup owns
// 32 MI x 32 NI outputs and its four wavefronts share k: wavefront w takes the k-groups (of 64) w, w + 4, ..., with a ring
// of two stages of its own in LDS, filled by global_load_lds as in the kernel above.  Nobody shares a stage, so there
// is no barrier in the loop: a wavefront waits for its own loads by count and keeps two groups in flight (three or four brought
// nothing: 197 x 768 x 3072 6.4 and 6.6 us with two and four, and they keep a second workgroup off the CU).  The four
// partial tiles are added through LDS in wavefront order (the sum over k has another order than in the tiled
// kernels, so which products come here depends on their size alone).
// What bounds it: the CU's path from L2 (about 100 GB/s of operands per CU; a 32 x 32 tile has no reuse to speak of),
// then launch and epilogue.  Chain of equal launches, tiled kernels -> here: 197 rows, 768 x 768 8.1 -> 4.0 us, 768 from
// 3072 21.0 -> 6.4, 2304 from 768 8.2 -> 5.2; 788 rows, 384 from 1536 12.6 -> 6.3; 1182 rows, 768 from 3072 21 -> 16.
// (Fragments straight from global memory, without LDS: 13.5 us for 197 x 768 x 3072; a load then touches 32 lines.)
// LNF: the folded LayerNorm; a wavefront adds up the rows of its k-groups from its fragments of A.
template <int MI, int NI, bool LNF>
__global__ __launch_bounds__(256, 1) void gemm_nt_few_kernel(BSR_HOT_PARAMS, GemmDesc g) {
  BSR_HOT_INTO(g);
  constexpr int NW = 4, NST = 2, BM = 32 * MI, BN = 32 * NI, LDP = BN + 4, LPT = 4 * (MI + NI), STAGE = LPT * 1024;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63, lr = lane & 31, lh = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ntm = (g.M + BM - 1) / BM;
  const int tile = xcd_remap(blockIdx.x, tiles);            // an XCD's range runs over the rows first: weights are read once
  const int m0 = (tile % ntm) * BM, n0 = (tile / ntm) * BN;
  const bf16* __restrict__ A = (const bf16*)g.A;
  const bf16* __restrict__ Bt = (const bf16*)g.B;
  unsigned char* ring = smem + wave * NST * STAGE;
  // load i fills tile rows 8 i .. 8 i + 7 (A rows first): lane (row lane / 8, slot lane % 8) fetches chunk slot ^ swz(row)
  unsigned off[LPT];
#pragma unroll
  for (int i = 0; i < LPT; ++i) {
    const int row = 8 * i + (lane >> 3), chunk = ((lane & 7) ^ swz(row)) * 8;
    off[i] = i < 4 * MI ? (unsigned)min(m0 + row, g.M - 1) * (unsigned)g.a_rs + chunk
                        : (unsigned)min(n0 + row - BM, g.N - 1) * (unsigned)g.b_cs + chunk;
  }
  auto issue = [&](int grp, int st) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < LPT; ++i)
      __builtin_amdgcn_global_load_lds(BSR_GLOBAL_PTR((i < 4 * MI ? A : Bt) + (size_t)grp * 64 + off[i]),
                                       BSR_LDS_VOID(ring + st * STAGE + i * 1024), 16, 0, 0);
  };
  f32x16 acc[MI][NI];
#pragma unroll
  for (int mi = 0; mi < MI; ++mi)
#pragma unroll
    for (int ni = 0; ni < NI; ++ni)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[mi][ni][r] = 0.f;
  float rsum[MI], rsq[MI];
#pragma unroll
  for (int mi = 0; mi < MI; ++mi) rsum[mi] = rsq[mi] = 0.f;
  const int sw = swz(lr), ng = g.K / 64;
  const int mine = ng > wave ? (ng - wave + NW - 1) / NW : 0;      // k-groups of this wavefront
  if (mine > 0) issue(wave, 0);
  if (mine > 1) issue(wave + NW, 1);
  // what the epilogue adds, asked for behind the first loads (as in EpiAhead above): thread tid finishes eight columns of rows tid / (BN / 8) + i * STEP
  constexpr int STEP = 256 / (BN / 8), ITEMS = (BM * BN / 8 + 255) / 256;
  const int erow = tid / (BN / 8), ecol = n0 + tid % (BN / 8) * 8;
  float bias[8], cs[8];
  Extra8 extra[ITEMS];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    bias[j] = g.bias && ecol < g.N ? g.bias[ecol + j] : 0.f;
    cs[j] = LNF && ecol < g.N ? g.ln_colsum[ecol + j] : 0.f;
  }
#pragma unroll
  for (int i = 0; i < ITEMS; ++i)
    if (erow + i * STEP < BM && m0 + erow + i * STEP < g.M && ecol < g.N) extra[i].fetch(g, m0 + erow + i * STEP, ecol);
  for (int i = 0; i < mine; ++i) {
    const int st = i & 1;
    if (i + 1 < mine) wait_vmcnt<LPT>();                           // the next group stays in flight
    else wait_vmcnt<0>();
    BSR_SCHED_FENCE();
    const unsigned char* s = ring + st * STAGE;
    bf16x8 fa[4][MI], fb[4][NI];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
#pragma unroll
      for (int mi = 0; mi < MI; ++mi) fa[ks][mi] = *(const bf16x8*)(s + (mi * 32 + lr) * 128 + (((ks * 2 + lh) ^ sw) << 4));
#pragma unroll
      for (int ni = 0; ni < NI; ++ni) fb[ks][ni] = *(const bf16x8*)(s + (BM + ni * 32 + lr) * 128 + (((ks * 2 + lh) ^ sw) << 4));
    }
    if (i + NST < mine) {
      wait_lgkmcnt0();                                             // the stage has been read: it can be filled again
      BSR_SCHED_FENCE();
      issue(wave + (i + NST) * NW, st);
    }
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
      for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
          acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[ks][mi], fb[ks][ni], acc[mi][ni], 0, 0, 0);
    if constexpr (LNF) {
      const bf16x2 ones = __builtin_bit_cast(bf16x2, 0x3f803f80u);
#pragma unroll
      for (int ks = 0; ks < 4; ++ks)
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
          for (int w = 0; w < 4; ++w) {
            unsigned word = __builtin_bit_cast(u32x4, fa[ks][mi])[w];
            asm("" : "+v"(word));                                  // (keeps the four words of a chunk apart, as above)
            const bf16x2 pr = __builtin_bit_cast(bf16x2, word);
            rsum[mi] = __builtin_amdgcn_fdot2_f32_bf16(pr, ones, rsum[mi], false);
            rsq[mi] = __builtin_amdgcn_fdot2_f32_bf16(pr, pr, rsq[mi], false);
          }
    }
  }
  __syncthreads();
  float* part = (float*)smem;
  float2* stat = (float2*)(part + NW * BM * LDP);                  // per wavefront and row: sum, sum of squares
  if constexpr (LNF) {
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) {
      rsum[mi] += __shfl_xor(rsum[mi], 32);
      rsq[mi] += __shfl_xor(rsq[mi], 32);
      if (lh == 0) stat[wave * BM + mi * 32 + lr] = make_float2(rsum[mi], rsq[mi]);
    }
  }
#pragma unroll
  for (int mi = 0; mi < MI; ++mi)
#pragma unroll
    for (int ni = 0; ni < NI; ++ni)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        part[(wave * BM + mi * 32 + 8 * (r >> 2) + 4 * lh + (r & 3)) * LDP + ni * 32 + lr] = acc[mi][ni][r];
  __syncthreads();
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    const int row = erow + i * STEP, m = m0 + row;
    if (row >= BM || m >= g.M || ecol >= g.N) continue;
    const float* p = part + row * LDP + ecol - n0;
    float v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = p[j];
#pragma unroll
    for (int w = 1; w < NW; ++w)
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] += p[w * BM * LDP + j];
    float2 ms = make_float2(0.f, 0.f);
    if constexpr (LNF) {
#pragma unroll
      for (int w = 0; w < NW; ++w) { ms.x += stat[w * BM + row].x; ms.y += stat[w * BM + row].y; }
      const float mean = ms.x / (float)g.K;
      ms = make_float2(mean, rsqrtf(fmaxf(ms.y / (float)g.K - mean * mean, 0.f) + g.ln_eps));
    }
    finish8(g, v, m, ecol, bias, cs, LNF ? &ms : nullptr, &extra[i]);
  }
}

template <int MI, int NI, bool LNF>
void launch_few_as(const GemmDesc& g, hipStream_t s) {
  constexpr size_t ring = (size_t)4 * 2 * 4 * (MI + NI) * 1024;
  constexpr size_t part = (size_t)4 * 32 * MI * ((32 * NI + 4) * sizeof(float) + sizeof(float2));
  constexpr size_t lds = ring > part ? ring : part;
  static bool attr_set = false;
  if (!attr_set) {
    (void)hipFuncSetAttribute((const void*)gemm_nt_few_kernel<MI, NI, LNF>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    attr_set = true;
  }
  const int tiles = ((g.M + 32 * MI - 1) / (32 * MI)) * ((g.N + 32 * NI - 1) / (32 * NI));
  gemm_nt_few_kernel<MI, NI, LNF><<<tiles, 256, lds, s>>>(BSR_HOT_ARGS(g, tiles), g);
}
template <int MI, int NI>
void launch_few(const GemmDesc& g, hipStream_t s) {
  if (g.ln_colsum) launch_few_as<MI, NI, true>(g, s);
  else launch_few_as<MI, NI, false>(g, s);
}
// 32 x 64 tiles are never ahead of both 64 x 32 and 64 x 64.
// c: modelled time of a product here, in microseconds, in the form of the tiled kernels' model: with t tiles, c0 +
// ceil(t / 256) (c1 + c2 K / 64) + t / 256 (c3 + c4 K / 64) + ceil(t / 512) (c5 + c6 K / 64), and t / 256 c7 where a GELU is applied.
// Constants fitted to chains of equal launches at 32 .. 2144 rows, N and K of 384 .. 3072 (108 products): the picks take 0.4 % longer than the
// fastest of the three.
// The other three are what the rule for coming here at all goes by (few_rows_shape): launch and epilogue, then ceil(t / 256) rounds of a
// start-up and the tile's operand bytes (within 15 % where this kernel is the faster one; its tiles would take 5.5 % longer than the fastest).
struct FewShape { int mi, ni; float c[8], launch_us, round_us, bytes_per_us; };
const FewShape kFewShapes[] = {{1, 1, {1.870f, 0.140f, 0.068f, 0.000f, 0.022f, 0.841f, 0.000f, 0.102f}, 2.6f, 0.5f, 105e3f},
                               {2, 1, {1.672f, 1.466f, 0.090f, 0.000f, 0.072f, 0.000f, 0.000f, 0.143f}, 2.8f, 0.5f, 103e3f},
                               {2, 2, {1.598f, 2.827f, 0.154f, 0.039f, 0.092f, 0.000f, 0.000f, 0.414f}, 3.3f, 1.0f, 65e3f}};

// The shape of this kernel for a product, or -1: not one it takes; *rule_us: the time that the rule compares
int few_pick(const GemmDesc& g, float* rule_us) {
  if (g.K % 64 || g.grp_off || !offsets_fit(g)) return -1;
  int pick = -1;
  float least = 0.f;
  for (int i = 0; i < 3; ++i) {
    const FewShape& f = kFewShapes[i];
    const int64_t tiles = (int64_t)((g.M + 32 * f.mi - 1) / (32 * f.mi)) * ((g.N + 32 * f.ni - 1) / (32 * f.ni));
    const float k = g.K / 64, w = (float)tiles / 256.f, rounds = (float)((tiles + 255) / 256);
    const float t = f.c[0] + rounds * (f.c[1] + f.c[2] * k) + w * (f.c[3] + f.c[4] * k + (g.act == ACT_NONE ? 0.f : f.c[7])) +
                    (float)((tiles + 511) / 512) * (f.c[5] + f.c[6] * k);
    const float r = f.launch_us + rounds * (f.round_us + 64.f * (f.mi + f.ni) * g.K / f.bytes_per_us);
    if (pick < 0 || t < least) { pick = i; least = t; }
    if (i == 0 || r < *rule_us) *rule_us = r;
  }
  return pick;
}
void launch_few(int pick, const GemmDesc& g, hipStream_t s) {
  if (pick == 0) launch_few<1, 1>(g, s);
  else if (pick == 1) launch_few<2, 1>(g, s);
  else launch_few<2, 2>(g, s);
}

// ------------------------------------------------------------------------------------------ TN
// Weight gradient dW[Mo,No] = sum_t X[t,Mo]^T dY[t,No] (Eq. 4): both operands have the contraction
// index t (tokens) as their row index, so an MFMA fragment (8 consecutive t for one column) is
// strided in memory.  The tiles are staged in LDS as they lie in memory - 64 token rows of 16-byte
// chunks - and the fragments are read with the LDS transpose read
// (ds_read_b64_tr_b16): within every 16 lanes, lane 4e+q passes the address of 4 columns of token
// row e, and lane j receives column j of the four rows, i.e. 4 consecutive tokens of one column.
// A fragment is two such reads (token rows r..r+3 and r+4..r+7).  One half-wave reads 4 rows x 64
// bytes; the 64-byte segments of a row are permuted by segment ^ (row & 3) so that those four land
// in four different bank groups (a row of 128 columns spans all 64 banks exactly once).
// Loads and arithmetic are two kinds of wavefront.  Four loaders fill a ring of NST stages with global_load_lds and wait
// for them by count; eight others only read fragments and multiply; one barrier per k-tile hands a landed stage over and a
// read one back.  A wavefront that did both would wait for every load in flight in front of each transpose read: the
// compiler cannot tell that such a read does not touch what a load is writing (measured so, 768 x 3072 over 25216 tokens:
// 167 us; register-staged 201; loaders of their own 141).  Two loaders are too few (154), a higher priority for them is worth
// up to 2 %.  What bounds it then is the path from L2 (64 bytes a clock into LDS) and, at many tokens, memory: the loads
// alone take 119 of those 141 us.
// The MFMA operands are swapped as in the direct-to-LDS NT kernel: accumulators hold transposed tiles.
// The tokens are cut into parts of kt_per k-tiles, by the sizes alone (tn_kt_per): each part is summed from zero and the parts
// are added up in ascending order, whichever workgroups they were summed by (bit-reproducible, no atomics).  A sum in parts is also the
// more precise one: over 6304 tokens dW is 2.4e-7 off its value in 64 bits (768 x 2304, three parts), summed in one chain 5.0e-7.
// A workgroup takes one part or, with 128 x 128 tiles, `run` of them in a row: the first one of a tile adds its parts up in
// registers, the others leave a partial each, and wavefronts of the next such launch add these to the first's.
// Bias gradient: the workgroups of the first row of tiles also multiply every dY fragment by an
// all-ones fragment, which leaves the column sums of dY (db = 1^T dY) in one more accumulator per
// 32 columns; they travel through the same partial / reduce path as dW.
#define BSR_LDS_PTR(T, p) ((T __attribute__((address_space(3)))*)(p))

constexpr int TN_LOADERS = 4, TN_THREADS = (8 + TN_LOADERS) * 64;

// What a weight gradient needs in a launch: its product, its parts, and the sums of the previous one.
struct TnArgs {
  GemmDesc g;
  float *partial, *bpartial;     // [1 + parts - run], null where a workgroup takes them all
  int kt_per;                    // k-tiles of a part
  int run;                       // parts of a workgroup
  int blocks;                    // tiles x runs (or groups)
  TnReduce red;                  // partials of an earlier launch to add up; splits == 0: none
};

// Workgroup lin of gx tiles x runs (grouped: x groups), tile fastest.
template <int BM, int BN, int WM, int WN, int NST>
__device__ __forceinline__ void tn_body(TnArgs a, int lin) {
  constexpr int NP = TN_LOADERS, NC = WM * WN;
  constexpr int TM = BM / WM, TN = BN / WN, MI = TM / 32, NI = TN / 32, NMF = MI * NI, NFR = MI + NI;
  constexpr int ABYTES = 64 * BM * 2, STAGE = (BM + BN) * 128;       // a stage: 64 token rows of A columns, then of B columns
  static_assert(BM % 128 == 0 && BN % 128 == 0, "the segment permutation needs a multiple of 4 segments per row");
  static_assert(NC == 8 && NMF >= 2 && NMF <= 16, "");
  constexpr bool RUNS = NMF == 2;                      // registers for a sum beside the one that is being taken
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  GemmDesc g = a.g;
  const int ntn = (g.N + BN - 1) / BN, ntm = (g.M + BM - 1) / BM, gx = ntm * ntn;
  const int tile = lin % gx, by = lin / gx;
  // an XCD's contiguous range of tiles runs along the side with fewer tiles first, so that it spans that side
  // and its L2 fetches the longer operand's token rows once instead of once per XCD
  const bool mfast = ntm < ntn;
  const int m0 = (mfast ? tile % ntm : tile / ntn) * BM, n0 = (mfast ? tile / ntm : tile % ntn) * BN;
  float *partial = a.partial, *bpartial = a.bpartial;
  int kt0 = by * a.run * a.kt_per, nk = min(a.run * a.kt_per, (g.K + BK - 1) / BK - kt0);
  if (g.grp_off) {
    // grouped form: by is the group; the contraction runs over its token rows only (perhaps none)
    const int r0 = g.grp_off[by], r1 = g.grp_off[by + 1];
    g.A = (const bf16*)g.A + (int64_t)r0 * g.a_cs;
    g.B = (const bf16*)g.B + (int64_t)r0 * g.b_rs;
    g.K = r1 - r0;
    g.C = (float*)g.C + (int64_t)by * g.c_gs;
    if (g.bsum) g.bsum += (int64_t)by * g.bsum_gs;
    kt0 = 0;
    nk = (g.K + BK - 1) / BK;
  }
  if (wave >= NC) {                                    // ---- loaders
    __builtin_amdgcn_s_setprio(3);
    constexpr int AR = 1024 / (BM * 2), BR = 1024 / (BN * 2);        // token rows one load instruction of a wavefront fills
    constexpr int AI = 64 / AR / NP, BI = 64 / BR / NP, LPP = AI + BI;   // load instructions of a loader per k-tile
    static_assert((AR == 4 || AR == 2) && (BR == 4 || BR == 2) && (NST - 1) * LPP <= 63, "vmcnt has 6 bits");
    const int pw = wave - NC;
    const bf16* X = (const bf16*)g.A + (int64_t)kt0 * BK * g.a_cs;     // [K tokens, Mo], row stride a_cs
    const bf16* Y = (const bf16*)g.B + (int64_t)kt0 * BK * g.b_rs;     // [K tokens, No], row stride b_rs
    const int rows = g.K - kt0 * BK;                                   // token rows from here on
    const int ra = lane / (BM / 8), pa = lane % (BM / 8), rb = lane / (BN / 8), pb = lane % (BN / 8);
    // LDS slot p of token row r holds the chunk whose segment is permuted to it (columns past the end repeat valid ones: never stored)
    auto chunk = [](int r, int p) { return ((((p >> 2) ^ (r & 3)) << 2) | (p & 3)) * 8; };
    auto acol = [&](int r) { return min(m0 + chunk(r, pa), g.M - 8); };
    auto bcol = [&](int r) { return min(n0 + chunk(r, pb), g.N - 8); };
    // instruction i of loader pw holds rows (i NP + pw) AR + ra: r & 3 takes one value for four rows an instruction; with
    // two it depends on the parity of pw (NP is even)
    const int64_t aoff = (int64_t)ra * g.a_cs + acol(AR == 2 ? 2 * (pw & 1) + ra : ra);
    const int64_t boff = (int64_t)rb * g.b_rs + bcol(BR == 2 ? 2 * (pw & 1) + rb : rb);
    auto issue = [&](int kt, int st) __attribute__((always_inline)) {
      unsigned char* d = smem + st * STAGE + pw * 1024;
      if ((kt + 1) * BK <= rows) {
        const bf16* xb = X + ((int64_t)kt * BK + pw * AR) * g.a_cs;
        const bf16* yb = Y + ((int64_t)kt * BK + pw * BR) * g.b_rs;
#pragma unroll
        for (int i = 0; i < AI; ++i, xb += (int64_t)AR * NP * g.a_cs)
          __builtin_amdgcn_global_load_lds(BSR_GLOBAL_PTR(xb + aoff), BSR_LDS_VOID(d + i * NP * 1024), 16, 0, 0);
#pragma unroll
        for (int i = 0; i < BI; ++i, yb += (int64_t)BR * NP * g.b_rs)
          __builtin_amdgcn_global_load_lds(BSR_GLOBAL_PTR(yb + boff), BSR_LDS_VOID(d + ABYTES + i * NP * 1024), 16, 0, 0);
      } else {                                         // the last tokens: rows past them repeat the last one (cleared below)
#pragma unroll 1
        for (int i = 0; i < AI; ++i) {
          const int r = (i * NP + pw) * AR + ra;
          __builtin_amdgcn_global_load_lds(BSR_GLOBAL_PTR(X + (int64_t)min(kt * BK + r, rows - 1) * g.a_cs + acol(r)),
                                           BSR_LDS_VOID(d + i * NP * 1024), 16, 0, 0);
        }
#pragma unroll 1
        for (int i = 0; i < BI; ++i) {
          const int r = (i * NP + pw) * BR + rb;
          __builtin_amdgcn_global_load_lds(BSR_GLOBAL_PTR(Y + (int64_t)min(kt * BK + r, rows - 1) * g.b_rs + bcol(r)),
                                           BSR_LDS_VOID(d + ABYTES + i * NP * 1024), 16, 0, 0);
        }
      }
    };
    // k-tile kt is in LDS, up to `later` k-tiles behind it may still be on their way; token rows past the last are zero
    auto landed = [&](int kt, int st, int later) __attribute__((always_inline)) {
      if (NST >= 4 && later >= 3) wait_vmcnt<(NST >= 4 ? 3 : 0) * LPP>();
      else if (NST >= 3 && later >= 2) wait_vmcnt<(NST >= 3 ? 2 : 0) * LPP>();
      else if (later >= 1) wait_vmcnt<LPP>();
      else wait_vmcnt<0>();
      const int valid = rows - kt * BK;
      if (kt == nk - 1 && valid < BK) {                // each loader clears what it loaded
        unsigned char* d = smem + st * STAGE + pw * 1024 + lane * 16;
        for (int i = 0; i < AI; ++i)
          if ((i * NP + pw) * AR + ra >= valid) *(u32x4*)(d + i * NP * 1024) = u32x4{0u, 0u, 0u, 0u};
        for (int i = 0; i < BI; ++i)
          if ((i * NP + pw) * BR + rb >= valid) *(u32x4*)(d + ABYTES + i * NP * 1024) = u32x4{0u, 0u, 0u, 0u};
        wait_lgkmcnt0();
      }
    };
    if (nk <= 0) return;
    for (int j = 0; j < NST && j < nk; ++j) issue(j, j);
    landed(0, 0, min(nk, NST) - 1);
    __builtin_amdgcn_s_barrier();
    for (int kt = 0, st = 0; kt < nk; ++kt) {
      const int stn = st + 1 == NST ? 0 : st + 1;
      if (kt + 1 < nk) landed(kt + 1, stn, min(nk - 2 - kt, NST - 2));
      __builtin_amdgcn_s_barrier();                    // k-tile kt has been read, k-tile kt + 1 may be
      if (kt + NST < nk) issue(kt + NST, st);
      st = stn;
    }
    return;
  }

  // ---- wavefronts that multiply
  const int wm = wave / WN, wn = wave % WN;
  f32x16 acc[MI][NI];
#pragma unroll
  for (int mi = 0; mi < MI; ++mi)
#pragma unroll
    for (int ni = 0; ni < NI; ++ni)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[mi][ni][r] = 0.f;

  // transpose-read coordinates of this lane: j = lane % 16 inside its block of 16 lanes, the block
  // covers columns cb*16 .. +16 of the 32-column fragment for k-group lh (tokens lh*8 .. +8 of a k-step);
  // fragments in the order A0, B0 .. B(NI-1), A1 .. A(MI-1) as in the NT kernel
  typedef short s16x4 __attribute__((ext_vector_type(4)));
  union Frag { bf16x8 v; s16x4 h[2]; };
  const int lh = lane >> 5, cb = (lane >> 4) & 1, rj = (lane & 15) >> 2;    // rj: token row inside a group of four (= row & 3)
  int offr[NFR];
  Frag fr[2][NFR];
#pragma unroll
  for (int j = 0; j < NFR; ++j) {
    const bool isA = j == 0 || j > NI;
    const int idx = j == 0 ? 0 : (j <= NI ? j - 1 : j - NI);
    const int o = ((isA ? wm * TM : wn * TN) + idx * 32 + cb * 16 + (lane & 3) * 4) * 2, q = o >> 4;
    offr[j] = (isA ? 0 : ABYTES) + (lh * 8 + rj) * (isA ? BM : BN) * 2 + ((((q >> 2) ^ rj) << 2) + (q & 3)) * 16 + (o & 15);
  }
  auto rd1 = [&](auto SET, auto J, int st, int ks) __attribute__((always_inline)) {
    constexpr int set = decltype(SET)::value, j = decltype(J)::value;
    constexpr int rowb = ((j == 0 || j > NI) ? BM : BN) * 2;
    const unsigned char* p = smem + st * STAGE + offr[j] + ks * 16 * rowb;       // and row + 4: both have (row & 3) == rj
    fr[set][j].h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(BSR_LDS_PTR(s16x4, p));
    fr[set][j].h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(BSR_LDS_PTR(s16x4, p + 4 * rowb));
  };
  const bool do_bsum = g.bsum && m0 == 0 && wm == 0;     // uniform over the wavefront
  f32x16 accb[NI];
  bf16x8 ones;
#pragma unroll
  for (int e = 0; e < 8; ++e) ones[e] = (bf16)1.0f;
#pragma unroll
  for (int ni = 0; ni < NI; ++ni)
#pragma unroll
    for (int r = 0; r < 16; ++r) accb[ni][r] = 0.f;
  auto mf1 = [&](auto SET, auto J) __attribute__((always_inline)) {
    constexpr int set = decltype(SET)::value, j = decltype(J)::value, mi = j / NI, ni = j % NI;
    constexpr int ja = mi == 0 ? 0 : NI + mi, jb = 1 + ni;
    acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[set][jb].v, fr[set][ja].v, acc[mi][ni], 0, 0, 0);
    if (mi == MI - 1 && do_bsum) accb[ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[set][jb].v, ones, accb[ni], 0, 0, 0);
  };
  auto kstep = [&](auto SET, int st, int ks) __attribute__((always_inline)) {
    constexpr int set = decltype(SET)::value, RPM = (NFR + NMF - 1) / NMF;
    sfor<NMF>([&](auto J) __attribute__((always_inline)) {
      constexpr int j = decltype(J)::value;
      mf1(IC<set>{}, J);
      sfor<RPM>([&](auto R) __attribute__((always_inline)) {
        constexpr int r = j * RPM + decltype(R)::value;
        if constexpr (r < NFR) rd1(IC<set ^ 1>{}, IC<r>{}, st, ks);
      });
      BSR_SCHED_FENCE();
    });
  };
  // the last k-step of a k-tile (fragments in set 1) with the barrier; behind it the first fragments of the next k-tile
  // are read (after the last one they are idle)
  auto klast = [&](int stn) __attribute__((always_inline)) {
    constexpr int PRE = NMF >= 16 ? 4 : (NMF >= 8 ? 2 : 1), POST = NMF - PRE, RPP = (NFR + POST - 1) / POST;
    sfor<PRE>([&](auto J) __attribute__((always_inline)) { mf1(IC<1>{}, J); BSR_SCHED_FENCE(); });
    wait_lgkmcnt0();                                   // this wavefront's reads of the stage are done
    __builtin_amdgcn_s_barrier();
    BSR_SCHED_FENCE();
    sfor<POST>([&](auto P) __attribute__((always_inline)) {
      constexpr int p = decltype(P)::value;
      mf1(IC<1>{}, IC<PRE + p>{});
      sfor<RPP>([&](auto R) __attribute__((always_inline)) {
        constexpr int r = p * RPP + decltype(R)::value;
        if constexpr (r < NFR) rd1(IC<0>{}, IC<r>{}, stn, 0);
      });
      BSR_SCHED_FENCE();
    });
  };
  auto store_bsum = [&](float* dst) __attribute__((always_inline)) {
    if (!do_bsum || (lane & 31) != 0) return;          // every column of accb holds the column sums
#pragma unroll
    for (int ni = 0; ni < NI; ++ni)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int col = n0 + wn * TN + ni * 32 + 8 * (r >> 2) + 4 * lh + (r & 3);
        if (col < g.N) dst[col] = accb[ni][r];
      }
  };
  int slot = by == 0 ? 0 : 1 + (by - 1) * a.run;       // partial of the part that is being summed
  // what the first workgroup of a tile has added up so far (-0 + x is x, whatever x)
  f32x16 sum[RUNS ? MI : 1][RUNS ? NI : 1], sumb[RUNS ? NI : 1];
  if constexpr (RUNS) {
#pragma unroll
    for (int ni = 0; ni < NI; ++ni)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        sumb[ni][r] = -0.f;
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) sum[mi][ni][r] = -0.f;
      }
  }
  // a part that is not this workgroup's last has been summed
  auto next_part = [&]() __attribute__((always_inline)) {
    if (by == 0) {
#pragma unroll
      for (int ni = 0; ni < NI; ++ni) {
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) sum[mi][ni] += acc[mi][ni];
        sumb[ni] += accb[ni];
      }
    } else {
      float* dst = partial + (int64_t)slot * g.M * g.N;
#pragma unroll
      for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int row = m0 + wm * TM + mi * 32 + (lane & 31), col = n0 + wn * TN + ni * 32 + 8 * q + 4 * lh;
            if (row < g.M && col < g.N)
              *(f32x4*)(dst + (int64_t)row * g.N + col) = f32x4{acc[mi][ni][4 * q], acc[mi][ni][4 * q + 1], acc[mi][ni][4 * q + 2], acc[mi][ni][4 * q + 3]};
          }
      if (bpartial) store_bsum(bpartial + (int64_t)slot * g.N);
      ++slot;
    }
#pragma unroll
    for (int ni = 0; ni < NI; ++ni)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        accb[ni][r] = 0.f;
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) acc[mi][ni][r] = 0.f;
      }
  };
  if (nk > 0) {
    __builtin_amdgcn_s_barrier();
    sfor<NFR>([&](auto J) __attribute__((always_inline)) { rd1(IC<0>{}, J, 0, 0); });
    for (int kt = 0, st = 0, left = a.kt_per; kt < nk; ++kt) {
      const int stn = st + 1 == NST ? 0 : st + 1;
      kstep(IC<0>{}, st, 1);
      kstep(IC<1>{}, st, 2);
      kstep(IC<0>{}, st, 3);
      klast(stn);
      st = stn;
      if constexpr (RUNS)
        if (--left == 0 && kt + 1 < nk) {
          next_part();
          left = a.kt_per;
        }
    }
  }
  if constexpr (RUNS)
    if (by == 0) {
#pragma unroll
      for (int ni = 0; ni < NI; ++ni) {
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) acc[mi][ni] = sum[mi][ni] + acc[mi][ni];
        accb[ni] = sumb[ni] + accb[ni];
      }
    }
  epilogue_f32<MI, NI>(partial ? partial + (int64_t)slot * g.M * g.N : (float*)g.C, partial ? g.N : g.ldc, g.M, g.N, acc, m0 + wm * TM,
                       n0 + wn * TN, lane, smem + wave * (32 * (TN * 4 + 16)));
  store_bsum(bpartial ? bpartial + (int64_t)slot * g.N : g.bsum);
}

// Tiles of a weight gradient: 128 x 128, four stages, or 256 x 128, three.
template <int T> struct TnTile;
template <> struct TnTile<0> { static constexpr int BM = 128, BN = 128, WM = 2, WN = 4, NST = 4; };
template <> struct TnTile<1> { static constexpr int BM = 256, BN = 128, WM = 4, WN = 2, NST = 3; };
template <class T> constexpr size_t tile_lds() { return (size_t)T::NST * (T::BM + T::BN) * 128; }
template <class T> constexpr size_t tile_patch_lds() { return (size_t)T::WM * T::WN * 32 * ((T::BN / T::WN) * 4 + 16); }

// k-tiles of a part and parts of a workgroup as one kernel argument (a workgroup takes at most 16 parts)
__host__ __device__ inline unsigned tn_pack(const TnArgs& a) { return (unsigned)a.kt_per | (unsigned)a.run << 26; }
__device__ inline void tn_unpack(TnArgs& a, unsigned parts) { a.kt_per = parts & 0x3ffffff; a.run = parts >> 26; }

// A weight gradient on its own.  Workgroups past the first `blocks` add up the partials of an earlier one.
template <int T>
__global__ __launch_bounds__(TN_THREADS, 1) void gemm_tn_kernel(const void* hA, const void* hB, int hM, int hN, int hK, unsigned ha_cs,
                                                                unsigned hb_rs, unsigned parts, int blocks, const int32_t* grp_off, TnArgs a) {
  using S = TnTile<T>;
  if ((int)blockIdx.x >= blocks) {
    const int64_t step = (int64_t)(gridDim.x - blocks) * TN_THREADS, items = splitk_reduce_items(a.red);
    for (int64_t it = (int64_t)(blockIdx.x - blocks) * TN_THREADS + threadIdx.x; it < items; it += step) splitk_reduce_item(a.red, it);
    return;
  }
  a.g.A = hA; a.g.B = hB; a.g.M = hM; a.g.N = hN; a.g.K = hK; a.g.a_cs = ha_cs; a.g.b_rs = hb_rs; a.g.grp_off = grp_off;
  tn_unpack(a, parts);
  tn_body<S::BM, S::BN, S::WM, S::WN, S::NST>(a, xcd_remap(blockIdx.x, blocks));
}

// Tiles of the input gradient in a launch that computes a layer's weight gradient as well.
template <int I> struct PairTile;
template <> struct PairTile<0> { static constexpr int BM = 128, BN = 64, WM = 2, WN = 2, NST = 4; };
template <> struct PairTile<1> { static constexpr int BM = 128, BN = 128, WM = 2, WN = 4, NST = 4; };
template <> struct PairTile<2> { static constexpr int BM = 192, BN = 128, WM = 2, WN = 4, NST = 3; };
template <> struct PairTile<3> { static constexpr int BM = 256, BN = 128, WM = 4, WN = 2, NST = 3; };

// Both gradients of a layer (Eq. 2 and Eq. 4): they read the same dy and neither reads what the other writes.  One
// workgroup per CU; the weight gradient's workgroups, which are the longest, come first, the input gradient's tiles fill
// the CUs they leave.  Its workgroups have wavefronts to spare: those add up the partials of the previous weight gradient.
// (Workgroups of their own for these sums hold a CU each: 768 x 768 over 2144 tokens took 1.24 times as long where they no longer
// fitted beside the tiles.)  Against the register-staged pair that this replaces, both gradients, calls in a row that add their partials up in a
// launch of their own: 2144 tokens 768 x 3072 43.6 -> 28.0 us, 3072 x 768 with GELU' 52.6 -> 38.0, 768 x 2304 41.8 -> 24.6; where the partials are
// most of it 768 x 768 21.6 -> 22.6, 384 x 1536 23.5 -> 22.9; 25216 tokens 768 x 3072 325 -> 238, 768 x 2304 247 -> 181; 1.18x over 112 shapes of
// 197 .. 25216 tokens (0.87 .. 1.71).
// dy [M, out], x [M, in] and the weight matrix [in, out]: dx = dy W^T and dW = x^T dy share sizes and dy, and the 14 dwords of arguments that
// come in registers (below: BSR_HOT_PARAMS) hold what both begin with.
template <int I, int T>
__global__ __launch_bounds__(TN_THREADS, 1) void gemm_pair_kernel(const void* dy, const void* w, const void* x, int M, int in, int out,
                                                                  unsigned dy_rs, unsigned w_rs, unsigned x_rs, unsigned parts, int tn_blocks,
                                                                  GemmDesc g, TnArgs a) {
  using N = PairTile<I>;
  using S = TnTile<T>;
  constexpr int NTHR = N::WM * N::WN * 64;
  if ((int)blockIdx.x < tn_blocks) {
    a.g.A = x; a.g.B = dy; a.g.M = in; a.g.N = out; a.g.K = M; a.g.a_cs = x_rs; a.g.b_rs = dy_rs; a.g.grp_off = nullptr;
    tn_unpack(a, parts);
    tn_body<S::BM, S::BN, S::WM, S::WN, S::NST>(a, xcd_remap(blockIdx.x, tn_blocks));
    return;
  }
  const int tile = blockIdx.x - tn_blocks, tiles = ((M + N::BM - 1) / N::BM) * ((in + N::BN - 1) / N::BN);
  if (threadIdx.x >= NTHR) {
    const int64_t items = a.red.splits > 0 ? splitk_reduce_items(a.red) : 0;
    for (int64_t it = (int64_t)tile * (TN_THREADS - NTHR) + threadIdx.x - NTHR; it < items; it += (int64_t)tiles * (TN_THREADS - NTHR))
      splitk_reduce_item(a.red, it);
    return;
  }
  g.A = dy; g.B = w; g.M = M; g.N = in; g.K = out; g.a_rs = dy_rs; g.b_cs = w_rs; g.grp_off = nullptr;
  ntd_body<N::BM, N::BN, N::WM, N::WN, N::NST>(g, xcd_remap(tile, tiles));
}

// the same reduction as a launch of its own
__global__ void splitk_reduce_kernel(TnReduce r) {
  const int64_t it = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (it < splitk_reduce_items(r)) splitk_reduce_item(r, it);
}

void launch_reduce(const TnReduce& r, hipStream_t s) {
  splitk_reduce_kernel<<<(unsigned)((splitk_reduce_items(r) + 255) / 256), 256, 0, s>>>(r);
}

bool is_tn(const GemmDesc& g) {
  return !g.in_f32 && g.out_f32 && g.a_rs == 1 && g.b_cs == 1 && g.M % 8 == 0 && g.N % 8 == 0 && g.M >= 8 &&
         g.N >= 8 && g.a_cs % 8 == 0 && g.b_rs % 8 == 0 && g.a_cs <= INT32_MAX && g.b_rs <= INT32_MAX && g.ldc % 8 == 0 && g.K > 0 && !g.res && g.act == ACT_NONE &&
         g.remap_np == 0 && (((uintptr_t)g.A | (uintptr_t)g.B | (uintptr_t)g.C) & 15) == 0;
}

// k-tiles of a part of a weight gradient's tokens: parts for 384 workgroups of 128 x 128 (512 from 96 k-tiles on), none
// below four k-tiles, at most 16, as many as the workspace has room for.  Sizes alone: it is the order of the sum.
int tn_kt_per(const GemmDesc& g, size_t room) {
  const int nk = (g.K + BK - 1) / BK;
  const int64_t tiles = (int64_t)((g.M + 127) / 128) * ((g.N + 127) / 128);
  const size_t per_part = (size_t)g.M * g.N + (g.bsum ? (size_t)g.N : 0);             // partial dW, then partial column sums
  const int parts = (int)std::min<int64_t>({(nk >= 96 ? 512 : 384) / tiles, nk / 4, (int64_t)std::min<size_t>(room / per_part, 16), 16});
  return parts > 1 ? (nk + parts - 1) / parts : nk;
}

// How many parts a workgroup of a weight gradient takes, its tile, and which tile its input gradient takes where nothing was
// measured: the combination that a model of the launch finishes first.  With one workgroup per CU a workgroup takes
// c0 + c1 k-tiles (an input gradient with GELU' gelu more; `partial` more for each partial sum that it leaves);
// the launch takes what list scheduling over 256 CUs takes (weight gradient first), a start, and the bytes of the partial
// sums.  Constants fitted to every combination on 112 layers (384 and 768 wide, 197 .. 25216 tokens, 1 .. 16 partials, launches in a
// row, one part a workgroup).  Steps with the parts of a workgroup forced to 1, 2, 3, 4 and all, and by the model, in us: ViT-B, 32 images
// 2320, 2256, 2226, 2231, 2241 and 2232, 128 images 5687, 5765, 5709, 5644, 5791 and 5633; DeiT-S, 32 images with AdamW 1348, 1308, 1290, 1300, 1370
// and 1271, 577 tokens 1740, 1715, 1709, 1716, 1831 and 1680.
struct PairCost { int bm, bn; float c0, c1, gelu; };
const PairCost kPairNt[] = {{128, 64, 2.00f, 0.365f, 2.88f}, {128, 128, 2.66f, 0.606f, 3.76f},
                            {192, 128, 4.43f, 0.621f, 4.70f}, {256, 128, 3.96f, 0.746f, 6.78f}};
struct TnCost { int bm, bn; float c0, c1, partial; };
const TnCost kTn[] = {{128, 128, 2.35f, 0.503f, 0.109f}, {256, 128, 3.57f, 0.864f, 0.359f}};
constexpr float PAIR_START_US = 2.08f, PAIR_PARTIAL_US = 2.02f;     // the latter per million floats of partial sums
constexpr int PAIR_CUS = 256;

// list scheduling: T workgroups of lt first, then N of ln
float pair_span(int64_t T, float lt, int64_t N, float ln) {
  const int64_t q = T / PAIR_CUS, r = T % PAIR_CUS;         // r CUs have q + 1 of the long ones, the others q
  const float base[2] = {q * lt, (q + 1) * lt}, least = (T * lt + N * ln) / PAIR_CUS;
  const int64_t cus[2] = {PAIR_CUS - r, r};
  float best = 0.f;
  bool found = N == 0;
  for (int f = 0; f < 2 && N > 0; ++f) {
    if (!cus[f]) continue;
    for (int64_t j = std::max<int64_t>(0, (int64_t)((least - base[f]) / ln)); ; ++j) {
      const float x = base[f] + j * ln;
      if (found && x >= best) break;
      const float other = x - base[1 - f];
      if (cus[f] * j + (other > 0.f ? cus[1 - f] * (int64_t)(other / ln + 1e-4f) : 0) >= N) { best = x; found = true; break; }
    }
  }
  return std::max(best, base[r > 0]);
}

struct TnSplit {
  int tile = 0, kt_per = 0, run = 1, nt = 1;     // tile of the weight gradient, k-tiles of a part, parts of a workgroup, tile of the input gradient
  int runs = 1, partials = 0;                    // workgroups of a tile, what they leave to be added up (0: nothing)
};
// floats of the split-K workspace that one launch may fill
size_t tn_room(size_t ws_floats, bool chained) { return chained ? (ws_floats / 2) & ~(size_t)3 : ws_floats; }

// nt: the input gradient of the same launch, or null
TnSplit tn_split(const GemmDesc* nt, const GemmDesc& g, size_t room) {
  TnSplit best;
  const int nk = (g.K + BK - 1) / BK, per = tn_kt_per(g, room), parts = (nk + per - 1) / per;
  float least = 0.f;
  bool any = false;
  for (int run = 1; run <= parts; ++run) {
    const int runs = (parts + run - 1) / run, partials = runs > 1 ? 1 + parts - run : 0;
    const float sums = PAIR_PARTIAL_US * partials * ((float)g.M * g.N * 1e-6f);
    for (int t = 0; t < (run == 1 ? 2 : 1); ++t) {
      const int64_t T = (int64_t)((g.M + kTn[t].bm - 1) / kTn[t].bm) * ((g.N + kTn[t].bn - 1) / kTn[t].bn) * runs;
      const float lt = kTn[t].c0 + kTn[t].c1 * per * run + kTn[t].partial * (runs > 1 ? run : 0);
      for (int i = 0; i < (nt ? 4 : 1); ++i) {
        if (nt && t == 1 && i < 2) continue;                // (small tiles beside large ones: never the fastest)
        const PairCost& c = kPairNt[i];
        const int64_t N = nt ? (int64_t)((nt->M + c.bm - 1) / c.bm) * ((nt->N + c.bn - 1) / c.bn) : 0;
        const float ln = c.c0 + c.c1 * (nt ? nt->K / BK : 0) + (nt && nt->act == ACT_GELU_BWD ? c.gelu : 0.f);
        const float us = PAIR_START_US + sums + pair_span(T, lt, N, ln);
        if (!any || us < least) { best = TnSplit{t, per, run, nt ? i : 1, runs, partials}; least = us; any = true; }
      }
    }
  }
  return best;
}

// Arguments of a weight-gradient launch: workspace half, the sums that wait in the chain (which it takes over) and the ones
// it leaves (in the chain, or in *mine without one).
TnArgs plan_tn(const GemmDesc& g, const TnSplit& sp, float* ws, size_t ws_floats, TnChain* chain, TnReduce* mine) {
  TnArgs a;
  a.g = g;
  a.partial = a.bpartial = nullptr;
  a.kt_per = sp.kt_per;
  a.run = sp.run;
  const int tiles = ((g.M + kTn[sp.tile].bm - 1) / kTn[sp.tile].bm) * ((g.N + kTn[sp.tile].bn - 1) / kTn[sp.tile].bn);
  a.blocks = tiles * (g.grp_off ? g.groups : sp.runs);      // (grouped: tiles x groups already fills the machine)
  *mine = TnReduce();
  if (chain) {       // this launch takes one half of the workspace, the pending reduction reads the other
    if (ws) ws += (size_t)chain->slot * tn_room(ws_floats, true);
    a.red = chain->pending;
    chain->pending = TnReduce();
  }
  if (sp.partials > 0) {
    const size_t mn = (size_t)g.M * g.N;
    a.partial = ws;
    a.bpartial = g.bsum ? ws + (size_t)sp.partials * mn : nullptr;
    mine->partial = ws; mine->n = (int64_t)mn; mine->splits = sp.partials; mine->out = (float*)g.C;
    mine->bpartial = a.bpartial; mine->nb = g.bsum ? g.N : 0; mine->bout = g.bsum;
    if (chain) {
      chain->pending = *mine;
      chain->slot ^= 1;
    }
  }
  return a;
}

template <int T>
void launch_tn_as(const TnArgs& a, hipStream_t s) {
  static bool attr_set = false;
  constexpr size_t lds = tile_lds<TnTile<T>>();
  static_assert(tile_patch_lds<TnTile<T>>() <= lds, "the epilogue patches live in the stage buffers");
  if (!attr_set) {
    (void)hipFuncSetAttribute((const void*)gemm_tn_kernel<T>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    attr_set = true;
  }
  // sums of an earlier launch: about four items per thread
  const int64_t per = (int64_t)TN_THREADS * 4;
  const int red = a.red.splits > 0 ? (int)std::min<int64_t>(512, (splitk_reduce_items(a.red) + per - 1) / per) : 0;
  gemm_tn_kernel<T><<<a.blocks + red, TN_THREADS, lds, s>>>(a.g.A, a.g.B, a.g.M, a.g.N, a.g.K, (unsigned)a.g.a_cs,
                                                            (unsigned)a.g.b_rs, tn_pack(a), a.blocks, a.g.grp_off, a);
}

void launch_tn(const GemmDesc& g, const TnSplit& sp, float* ws, size_t ws_floats, hipStream_t s, TnChain* chain) {
  TnReduce mine;
  const TnArgs a = plan_tn(g, sp, ws, ws_floats, chain, &mine);
  if (sp.tile) launch_tn_as<1>(a, s);
  else launch_tn_as<0>(a, s);
  if (!chain && mine.splits > 0) launch_reduce(mine, s);
}

template <int I, int T>
void launch_pair_as(const GemmDesc& g, const TnArgs& a, hipStream_t s) {
  using N = PairTile<I>;
  static bool attr_set = false;
  constexpr size_t lds = tile_lds<N>() > tile_lds<TnTile<T>>() ? tile_lds<N>() : tile_lds<TnTile<T>>();
  static_assert(tile_patch_lds<N>() <= lds && tile_patch_lds<TnTile<T>>() <= lds, "the epilogue patches live in the stage buffers");
  if (!attr_set) {
    (void)hipFuncSetAttribute((const void*)gemm_pair_kernel<I, T>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    attr_set = true;
  }
  const int tiles = ((g.M + N::BM - 1) / N::BM) * ((g.N + N::BN - 1) / N::BN);
  gemm_pair_kernel<I, T><<<a.blocks + tiles, TN_THREADS, lds, s>>>(g.A, g.B, a.g.A, g.M, g.N, g.K, (unsigned)g.a_rs,
                                                               (unsigned)g.b_cs, (unsigned)a.g.a_cs, tn_pack(a), a.blocks, g, a);
}
template <int I>
void launch_pair(const GemmDesc& g, const GemmDesc& t, const TnSplit& sp, float* ws, size_t ws_floats, hipStream_t s, TnChain* chain) {
  TnReduce mine;
  const TnArgs a = plan_tn(t, sp, ws, ws_floats, chain, &mine);
  if (sp.tile) launch_pair_as<I, 1>(g, a, s);
  else launch_pair_as<I, 0>(g, a, s);
  if (!chain && mine.splits > 0) launch_reduce(mine, s);
}

bool is_nt(const GemmDesc& g) {
  return !g.in_f32 && g.a_cs == 1 && g.b_rs == 1 && g.K % 8 == 0 && g.a_rs % 8 == 0 && g.b_cs % 8 == 0 &&
         g.N % 8 == 0 && g.ldc % 8 == 0 && g.ldr % 8 == 0 && (((uintptr_t)g.A | (uintptr_t)g.B | (uintptr_t)g.C) & 15) == 0 &&
         (((uintptr_t)g.aux | (uintptr_t)g.res) & 15) == 0 && g.M > 0 && g.N > 0 && g.K > 0;
}

}  // namespace

// two halves (a launch writes one while the previous launch's partials are added up from the other), each
// with room for 8 partial copies of the largest weight gradient of a block ([D,3D] or [D,F]) and of its
// bias gradient (16 for the smaller matrices, which split further)
size_t gemm_splitk_ws_floats(int dim, int mlp_hidden) {
  return 2 * ((size_t)8 * std::max((size_t)3 * dim * dim, (size_t)dim * mlp_hidden) +
              (size_t)16 * std::max(3 * dim, mlp_hidden));
}

bool gemm_mfma_supported(const GemmDesc& g) { return is_nt(g) || is_tn(g); }

// Tile choice.  What bounds these kernels on a CU is operand delivery, not the matrix cores: LDS
// takes writes at about 64 bytes per clock, so a k-tile of a BM x BN block tile costs 2 (BM + BN)
// clocks of LDS writes (plus the fragment reads) against BM * BN / 32 clocks of MFMA work.  Only
// 256 x 256 tiles keep that ratio well below one, but at M = 2144 .. 6304 rows they leave most CUs
// without a tile, so each launch takes the shape that a model predicts to be fastest (below), or the one a context
// has measured to be (bsr_autotune).  Every shape accumulates an output element over k in the same order, so the choice
// never changes a result.
static const int kNtShapes[] = {
    // staged through registers; what folds a LayerNorm or has a ragged K has these only
    256128, 128128, 192128, 160256, 256256, 128064, 64128,
    3128064,                              // with deeper register prefetch (id = PF * 1000000 + shape)
    // operands straight into LDS (id = 7000000 + shape, 8000000 + shape with one stage more; K a multiple of 64, no
    // folded LayerNorm: a launch outside that takes the model's shape instead)
    7256256, 7320256, 7192256, 7256192, 7256128, 7128256, 7192128, 7128128, 7128064, 7064128, 7096128, 8192128, 8128128,
};
// ids that callers may still hold, of register-staged shapes that no product was fastest on: they take the model's shape
static const int kNtRetired[] = {96128, 128256, 192256, 256064, 96256, 3064128, 2192128, 2256128, 2128128};
static bool is_retired(int id) { return std::find(std::begin(kNtRetired), std::end(kNtRetired), id) != std::end(kNtRetired); }
// stages of the direct-to-LDS shapes (0: not one of them)
static int ntd_stages(int id) {
  switch (id) {
    case 7256256: case 7320256: case 7192256: case 7256192: case 7192128: case 7128128: return 2;
    case 7256128: case 7128256: case 7128064: case 7064128: case 7096128: case 8192128: case 8128128: return 3;
    default: return 0;
  }
}

// The model: with t tiles, time = c0 + ceil(t / 256) (c1 + c2 K / 64) + t / 256 (c3 + c4 K / 64) + ceil(t / 512) (c5 + c6 K / 64)
// microseconds, and where a GELU or GELU' is applied ceil(t / 256) c7 + t / 256 c8 more: a fixed part, rounds of one workgroup per CU, what scales with
// the work, rounds of two per CU.  From MANY_RESULTS on a GELU beside which its input is stored takes ceil(t / 256) c9 instead of those (fitted to 318 products
// with every epilogue): there the two streams of results count, which larger tiles overlap better.  The line is where nothing beyond it loses; it is measured,
// not derived.  Steps with all blocks trained at the numbers of images where c9 takes another tile, c7 and c8 -> c9 (runs of one side differ by 0.5 %):
//   37.7 M results and more: 384 wide 125, 128, 160, 192, 256 images 0.991 .. 0.997, 512 wide 112, 120, 144, 160, 192, 256 images 0.984 .. 0.995,
//     768 wide 80, 96, 128, 160, 192 0.989 .. 0.994, 1024 wide 56, 72, 96, 112 0.984 .. 0.994
//   fewer: 384 wide 16 .. 103 images 0.993 .. 1.008, 512 wide 16 .. 77 0.994 .. 1.011, 768 wide 12 .. 51 0.986 .. 1.005, 56 .. 62 1.002 .. 1.012,
//     1024 wide 22 .. 45 0.991 .. 1.002 (36 steps, 0.999 on average)
// (A constant of the same kind for the GELU' changed 5 of 805 choices at 3072 x 768 and none at 1536 x 384 and 2048 x 512; steps with and without it 1.000.)
constexpr int64_t MANY_RESULTS = 36 << 20;
struct NtModel { int id, bm, bn; float c[10]; };
// Direct-to-LDS shapes: constants fitted to chains of equal launches over twelve weight matrices (88 products of 400 .. 25216
// rows; 384, 768, 1152, 1536, 2304 and 3072 columns).  Of 32 shapes measured there these nine lose 0.8 %, and the model's
// picks among them 1.2 %, to the fastest of all; the best of the shapes before them (four-wavefront and register-staged
// ones) took 6.5 % longer, the model's picks of those 14 %.  At other widths the model extrapolates, and tuning is the way to know.
const NtModel kNtModel[] = {
    {7128064, 128, 64, {2.231f, 0.226f, 0.225f, 0.244f, 0.063f, 1.485f, 0.040f, 1.032f, 0.000f, 0.514f}},
    {7192128, 192, 128, {3.692f, 0.495f, 0.423f, 1.425f, 0.145f, 0.000f, 0.241f, 2.731f, 0.000f, 2.115f}},
    {8128128, 128, 128, {1.293f, 2.977f, 0.363f, 0.000f, 0.181f, 0.000f, 0.000f, 1.970f, 0.623f, 1.448f}},
    {7128128, 128, 128, {2.632f, 0.784f, 0.200f, 0.475f, 0.149f, 0.273f, 0.363f, 1.768f, 0.000f, 1.302f}},
    {7320256, 320, 256, {0.696f, 7.695f, 0.752f, 0.000f, 1.252f, 1.771f, 0.190f, 10.720f, 0.381f, 6.316f}},
    {8192128, 192, 128, {1.428f, 3.720f, 0.438f, 0.000f, 0.294f, 0.000f, 0.000f, 2.450f, 1.429f, 2.910f}},
    {7192256, 192, 256, {1.340f, 5.269f, 0.721f, 0.000f, 0.597f, 0.321f, 0.000f, 6.615f, 0.367f, 3.911f}},
    {7256256, 256, 256, {0.390f, 6.475f, 0.912f, 0.000f, 0.791f, 1.970f, 0.000f, 7.088f, 1.735f, 3.884f}},
    {7256128, 256, 128, {0.000f, 4.160f, 0.564f, 0.268f, 0.342f, 1.936f, 0.000f, 3.777f, 0.839f, 2.225f}},
};
// Fitted to every shape forced in turn on the launches of ViT-B and DeiT-S steps (436 launches, event-bracketed, in their place
// in the step, the event pair included).  The register-staged ones, which come first, are picked from for products that only they
// take; all of them together are what the rule for products of few rows takes a tiled launch in a step for.
const NtModel kNtStepModel[] = {
    {64128, 64, 128, {6.508f, 0.000f, 0.142f, 1.061f, 0.000f, 0.000f, 0.353f, 0.f, 0.f}},
    {192128, 192, 128, {7.783f, 1.559f, 0.501f, 1.705f, 0.104f, 0.000f, 0.182f, 0.f, 0.f}},
    {256128, 256, 128, {3.608f, 3.854f, 0.664f, 2.056f, 0.342f, 2.154f, 0.001f, 0.f, 0.f}},
    {3128064, 128, 64, {6.542f, 0.794f, 0.173f, 0.773f, 0.052f, 0.000f, 0.222f, 0.f, 0.f}},
    {7256256, 256, 256, {0.000f, 8.827f, 1.173f, 1.403f, 0.332f, 5.356f, 0.142f, 0.f, 0.f}},
    {7320256, 320, 256, {10.479f, 4.369f, 1.469f, 3.163f, 0.515f, 0.945f, 0.009f, 0.f, 0.f}},
};
constexpr float EVENTS_US = 4.5f;      // the part of their c0 that a launch inside a chain does not take (the event pair)

// the fastest by a table of models, and the time it gives it.  (With the LayerNorm folded in, 64 columns per tile would
// double its dot instructions per MFMA.)
template <int N>
static int model_pick(const NtModel (&table)[N], const GemmDesc& g, bool direct_ok, float* us_out) {
  int pick = 0;
  const bool stored = g.act == ACT_GELU && g.aux && (int64_t)g.M * g.N >= MANY_RESULTS;
  const float k = (float)((g.K + BK - 1) / BK), gelu = g.act != ACT_NONE && !stored ? 1.f : 0.f;
  for (const NtModel& e : table) {
    if ((ntd_stages(e.id) && !direct_ok) || (g.ln_colsum && e.bn < 128)) continue;
    // (a group ends in a partial row tile: half a tile each)
    const int64_t t = (int64_t)((g.M + e.bm - 1) / e.bm + (g.grp_off ? g.groups / 2 : 0)) * ((g.N + e.bn - 1) / e.bn);
    const float r1 = (float)((t + 255) / 256), w = (float)t / 256.f, r2 = (float)((t + 511) / 512);
    const float us = e.c[0] + r1 * (e.c[1] + e.c[2] * k + e.c[7] * gelu + (stored ? e.c[9] : 0.f)) + w * (e.c[3] + e.c[4] * k + e.c[8] * gelu) +
                     r2 * (e.c[5] + e.c[6] * k);
    if (!pick || us < *us_out) { pick = e.id; *us_out = us; }
  }
  return pick;
}
static int nt_pick(const GemmDesc& g) {
  float us = 0.f;
  return is_ntd(g) ? model_pick(kNtModel, g, true, &us) : model_pick(kNtStepModel, g, false, &us);
}
size_t gemm_nt_tile_lds_bytes(int id) {
  const int bm = id % 1000000 / 1000, bn = id % 1000, nst = ntd_stages(id);
  return (size_t)(nst ? nst : 2) * (bm + bn) * BK * sizeof(bf16);
}
int gemm_nt_tile_count() { return (int)(sizeof(kNtShapes) / sizeof(kNtShapes[0])); }
int gemm_nt_tile_id(int i) { return kNtShapes[i]; }
bool gemm_nt_tile_known(int id) { return id == 0 || std::find(std::begin(kNtShapes), std::end(kNtShapes), id) != std::end(kNtShapes) || is_retired(id); }
bool gemm_nt_tile_is_free(const GemmDesc& g) { return is_nt(g) && !g.grp_off; }

// The one rule that sends a product to the kernel for few rows: the shape of that kernel, or -1 for the tiled ones.  It
// looks at the product's sizes, and at whether the launch could carry the layer's weight gradient as well (tiled kernels
// do that in one launch; here it costs another one), and at nothing else: the kernel for few rows adds over k in another
// order, so with the tile choice in the rule, tuning would change bits, and so does every shift of the line itself.
// A product goes there when it leads clearly over the tiled kernels as they run in a step, where every launch follows another
// kernel: near-ties went to the tiled ones there.  (A line without that lead, between the models fitted to chains of equal launches, came
// to 1.000x over 20 steps, 0.984 .. 1.019, and moved every gradient behind a product that changed sides by up to 1 %.)
constexpr float FEW_LEAD = 0.8f, TILED_LAUNCH_US = 2.6f;      // the latter: the launch that a weight gradient carried along saves
static int few_rows_shape(const GemmDesc& g, bool carries_wgrad) {
  float few_us = 0.f, tiled_us = 0.f;
  const int few = few_pick(g, &few_us);
  if (few < 0) return -1;
  model_pick(kNtStepModel, g, is_ntd(g), &tiled_us);
  return few_us < FEW_LEAD * (tiled_us - EVENTS_US - (carries_wgrad ? TILED_LAUNCH_US : 0.f)) ? few : -1;
}
// the two gradients of one layer: one dy, sizes that match
static bool one_layer(const GemmDesc& nt, const GemmDesc& tn) {
  return nt.A == tn.B && nt.a_rs == tn.b_rs && nt.M == tn.K && nt.N == tn.M && nt.K == tn.N && (int64_t)tn.K * tn.a_cs <= (int64_t)UINT32_MAX;
}
static bool can_pair(const GemmDesc& nt, const GemmDesc& tn) {
  return is_nt(nt) && is_ntd(nt) && !nt.grp_off && is_tn(tn) && !tn.grp_off && one_layer(nt, tn);
}

// Tile of the input gradient (index into kPairNt) in a layer's backward launch that is asked to take a shape; -1: the joint kernel
// has no such tile, two launches.  Several ids name one tile here: loads are straight into LDS whatever the id says, in one depth.
static int joint_tile(int tile, const TnSplit& pair) {
  if (!tile || is_retired(tile)) return pair.nt;
  for (int i = 0; i < 4; ++i)
    if (tile % 1000000 == 1000 * kPairNt[i].bm + kPairNt[i].bn) return i;
  return -1;
}
// Shape of a product on its own that is asked to take a shape: the model's for 0, for an id that was a shape once and for a shape that
// cannot take the product.
static int nt_tile(const GemmDesc& g, int tile) {
  if (tile >= APART_ID) tile -= APART_ID;
  return !tile || is_retired(tile) || (ntd_stages(tile) && !is_ntd(g)) ? nt_pick(g) : tile;
}
// Whether a layer's two gradients, with no shape asked for, go out one after the other: an input gradient with GELU' and many rows.  A joint
// launch has one workgroup a CU, so nothing covers a tile's epilogue, and a GELU' doubles that; on its own such a product takes larger tiles, or two
// workgroups a CU, and pays a launch and a second drain of the CUs for it.  Trained part of steps with all 12 blocks trained, joint -> apart, both forced:
//   3072 x 768:  3940 .. 9456 rows +0.5 .. +2.2 %, 10244 .. 13002 -2.9 .. +0.6 % (-1.2 on average), 13396 .. 25216 -1.9 .. +0.1 % (-1.0)
//   4096 x 1024: 6304 .. 19700 -0.8 .. +0.3 %
//   1536 x 384:  6304, 7880 +2.1, +1.0 %, 9456 .. 13002 -1.8 .. +1.2 % (mixed), 13396 .. 25216 -2.9 .. -1.9 %
//   2048 x 512:  9456 .. 12608 +0.2 .. +1.0 %, 14184 .. 25216 -1.7 .. +0.6 % (-0.8)
//   768 x 768, 1536 x 768, 3072 x 384: 9456, 12608 -1.5 .. +1.4 %, 14184 .. 25216 -3.0 .. +0.1 % (-1.3)
//   384 x 384, 768 x 192: 9456 .. 39400 +0.2 .. +3.7 %: too little to multiply for a second launch
// So there is a line for large matrices and one for smaller ones, each where nothing beyond it loses more than the runs differ by (0.6 %).
// (The two models' times do not draw this line: both leave out what launches lose to each other, and their rounds of tiles make it jump.)
static bool apart(const GemmDesc& nt) {
  const int64_t weights = (int64_t)nt.N * nt.K;
  return nt.act == ACT_GELU_BWD && weights >= 512 * 1024 && nt.M >= (weights >= 2048 * 1024 ? 10240 : 13312);
}
// whether they do when `tile` is asked for
static bool goes_apart(const GemmDesc& nt, int tile) { return tile >= APART_ID || ((!tile || is_retired(tile)) && apart(nt)); }
int gemm_nt_runs_tile(const GemmDesc& g, const GemmDesc* wgrad, size_t splitk_ws_floats, bool chained, int tile) {
  const int few = few_rows_shape(g, wgrad != nullptr);
  if (few >= 0) return FEW_ROWS_ID + 32000 * kFewShapes[few].mi + 32 * kFewShapes[few].ni;
  const int alone = nt_tile(g, tile);
  if (!wgrad || !can_pair(g, *wgrad)) return alone;
  const TnSplit split = tn_split(&g, *wgrad, tn_room(splitk_ws_floats, chained));
  if (goes_apart(g, tile)) return joint_tile(alone, split) < 0 ? alone : APART_ID + alone;
  const int i = joint_tile(tile, split);
  return i < 0 ? alone : 7000000 + 1000 * kPairNt[i].bm + kPairNt[i].bn;
}

TnReduce gemm_tn_take(TnChain* chain) {
  const TnReduce r = chain->pending;
  chain->pending = TnReduce();
  return r;
}

// The tiled kernels, in the shape asked for or, for 0 and for a shape that cannot take the product, the model's.
static void nt_tiled(const GemmDesc& g, hipStream_t s, int tile) {
  switch (nt_tile(g, g.grp_off ? 0 : tile)) {
    case 7256256: launch_ntd<256, 256, 2, 4, 2>(g, s); break;
    case 7320256: launch_ntd<320, 256, 2, 4, 2>(g, s); break;
    case 7192256: launch_ntd<192, 256, 2, 4, 2>(g, s); break;
    case 7256192: launch_ntd<256, 192, 4, 2, 2>(g, s); break;
    case 7256128: launch_ntd<256, 128, 4, 2, 3>(g, s); break;
    case 7128256: launch_ntd<128, 256, 2, 4, 3>(g, s); break;
    case 7192128: launch_ntd<192, 128, 2, 4, 2>(g, s); break;
    case 8192128: launch_ntd<192, 128, 2, 4, 3>(g, s); break;
    case 7128128: launch_ntd<128, 128, 2, 4, 2>(g, s); break;
    case 8128128: launch_ntd<128, 128, 2, 4, 3>(g, s); break;
    case 7128064: launch_ntd<128, 64, 2, 2, 3>(g, s); break;
    case 7064128: launch_ntd<64, 128, 2, 2, 3>(g, s); break;
    case 7096128: launch_ntd<96, 128, 1, 4, 3>(g, s); break;
    case 256256: launch_nt<256, 256, 2, 4>(g, s); break;
    case 256128: launch_nt<256, 128, 4, 4>(g, s); break;
    case 192128: launch_nt<192, 128, 2, 4>(g, s); break;
    case 160256: launch_nt<160, 256, 1, 8>(g, s); break;
    case 128064: launch_nt<128, 64, 4, 2>(g, s); break;
    case 64128: launch_nt<64, 128, 2, 4>(g, s); break;
    case 3128064: launch_nt<128, 64, 4, 2, 3>(g, s); break;
    default: launch_nt<128, 128, 4, 2>(g, s); break;
  }
}

void gemm_mfma(const GemmDesc& g, float* splitk_ws, size_t splitk_ws_floats, hipStream_t s, int tile, TnChain* chain) {
  if (is_tn(g)) {
    TnSplit split;
    if (g.grp_off) split.kt_per = (g.K + BK - 1) / BK;     // (all tokens of a group in one part)
    else split = tn_split(nullptr, g, tn_room(splitk_ws ? splitk_ws_floats : 0, chain != nullptr));
    launch_tn(g, split, splitk_ws, splitk_ws_floats, s, chain);
    return;
  }
  const int few = few_rows_shape(g, false);
  if (few >= 0) launch_few(few, g, s);
  else nt_tiled(g, s, tile);
}

// The input gradient (NT) and the weight gradient (TN) of one layer: one launch, unless the tile asked for is none of
// the shapes that the joint kernel has.  Which kernel multiplies, and which tokens are summed together, does not depend
// on the tile.
void gemm_mfma_pair(const GemmDesc& nt, const GemmDesc& tn, float* splitk_ws, size_t splitk_ws_floats, hipStream_t s,
                    int tile, TnChain* chain) {
  const int few = few_rows_shape(nt, true);
  if (few >= 0) {
    launch_few(few, nt, s);
    gemm_mfma(tn, splitk_ws, splitk_ws_floats, s, 0, chain);
    return;
  }
  const size_t room = tn_room(splitk_ws ? splitk_ws_floats : 0, chain != nullptr);
  if (can_pair(nt, tn) && !goes_apart(nt, tile)) {
    const TnSplit split = tn_split(&nt, tn, room);
    switch (joint_tile(tile, split)) {
      case 0: launch_pair<0>(nt, tn, split, splitk_ws, splitk_ws_floats, s, chain); return;
      case 1: launch_pair<1>(nt, tn, split, splitk_ws, splitk_ws_floats, s, chain); return;
      case 2: launch_pair<2>(nt, tn, split, splitk_ws, splitk_ws_floats, s, chain); return;
      case 3: launch_pair<3>(nt, tn, split, splitk_ws, splitk_ws_floats, s, chain); return;
      default: break;
    }
  }
  nt_tiled(nt, s, tile);                 // (not gemm_mfma: its rule is that of a product on its own)
  if (is_tn(tn)) launch_tn(tn, tn_split(nullptr, tn, room), splitk_ws, splitk_ws_floats, s, chain);
  else gemm_mfma(tn, splitk_ws, splitk_ws_floats, s, 0, chain);
}

}  // namespace bsr
