// fp32 GEMMs on the matrix cores (v_mfma_f32_32x32x2_f32: IEEE fp32 multiply-adds, 157 TFLOP/s on the chip),
// the products of the fp32 mode: forward, input gradient and weight gradient of every linear layer.
//
// What bounds it: the matrix cores.  A 32 x 32 x 2 MFMA takes 64 clocks and two floats per lane, so the LDS and L2
// traffic of even a 32 x 32 block tile fits beside it, and the choice of the block tile is about filling 256 CUs:
// at the sizes of this mode (M = 130 .. 1576 token rows) 128 x 128 tiles leave most CUs idle.  Three block tiles,
// picked by f32_pick below: 128 x 128 (4 wavefronts of 64 x 64), 64 x 64 (8 wavefronts: 4 quadrants x 2 halves of
// every k-tile) and 32 x 32 (8 wavefronts, each an eighth of every k-tile); the partial sums of the wavefronts that
// share a tile are added through LDS in a fixed order (bit-reproducible).
//
// Measured, DeiT-S step of 8 images: the products 11.5 ms as vector-unit kernels, 1.4 ms here (81 launches; 0.41 ms is
// what a large fp32 product on this chip would take); one 192-wide block of 130 rows: 60 -> 4.5 .. 7.7 us a product.
//
// The contraction index of an MFMA is a dummy: MFMA j of a group of 8 uses k = 4 h + j for wave half h, so a lane's
// four operands of four MFMAs are four consecutive floats.  An operand whose k is contiguous in memory is staged as
// it lies, rows of KT floats (+4: the 16-byte reads of 16 rows then hit every bank once), and read with one 16-byte
// LDS read per four MFMAs; an operand whose row index is contiguous is staged [k][row] (+8 per k-row: the two wave
// halves, four k-rows apart, hit different banks) and read with four 4-byte reads.
#include <algorithm>

#include "bsr_internal.h"

namespace bsr {

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ inline float gelu_f(float u) { return 0.5f * u * (1.0f + erff(u * 0.70710678118654752f)); }
__device__ inline float gelu_grad_f(float u) {
  const float cdf = 0.5f * (1.0f + erff(u * 0.70710678118654752f));
  return cdf + u * (expf(-0.5f * u * u) * 0.39894228040143268f);
}

// consecutive workgroups go to the 8 XCDs in turn: give each XCD a contiguous range of tiles
__device__ inline int xcd_range(int pid, int n) {
  const int base = n / 8, rem = n % 8, x = pid % 8;
  return x * base + min(x, rem) + pid / 8;
}

// k-tile: long where the wavefronts share it, since a tile that is alone on its CU is done with 32 k long before the
// next loads return (64 x 64 tiles at M = 1576, K = 384: 30 us with k-tiles of 32 fetched one ahead)
__host__ __device__ constexpr int f32_kt(int wk) { return wk == 1 ? 32 : wk == 2 ? 64 : 128; }

// One operand's tile in LDS: R rows (of the output index) x KT; KC: k contiguous in memory
template <int R, int KT, bool KC, int NT>
struct Tile {
  static constexpr int LD = KC ? KT + 4 : R + 8;                 // floats per LDS row
  static constexpr int FLOATS = KC ? R * LD : KT * LD;
  static constexpr int CPR = (KC ? KT : R) / 4;                  // 16-byte chunks per memory row
  static constexpr int NCH = R * KT / 4 / NT;                    // chunks per thread
  static_assert(R * KT / 4 % NT == 0 && NCH >= 1, "every thread carries whole chunks");
  f32x4 v[NCH];
  // p: operand, ld: floats between memory rows, r0: first output row of the tile, rows / K: extents
  __device__ __forceinline__ void fetch(const float* __restrict__ p, int64_t ld, int r0, int rows, int k0, int K, int tid) {
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      const int c = tid + NT * i, a = c / CPR, q = (c % CPR) * 4;
      const int r = KC ? r0 + a : r0 + q, k = KC ? k0 + q : k0 + a;
      // rows past the end repeat valid ones (never stored); k past the end is zero
      const float* src = KC ? p + (int64_t)min(r, rows - 1) * ld + min(k, K - 4) : p + (int64_t)min(k, K - 1) * ld + min(r, rows - 4);
      v[i] = *(const f32x4*)src;
      if (k >= K) v[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
  }
  __device__ __forceinline__ void stash(float* s, int tid) const {
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      const int c = tid + NT * i;
      *(f32x4*)(s + (c / CPR) * LD + (c % CPR) * 4) = v[i];
    }
  }
  // four consecutive k of output row r: k-group grp of 8, wave half h
  __device__ static __forceinline__ f32x4 frag(const float* s, int r, int grp, int h) {
    const int k = grp * 8 + h * 4;
    if constexpr (KC) {
      return *(const f32x4*)(s + r * LD + k);
    } else {
      f32x4 f;
#pragma unroll
      for (int j = 0; j < 4; ++j) f[j] = s[(k + j) * LD + r];
      return f;
    }
  }
};

template <int BM, int BN, int WM, int WN, int WK, bool AK, bool BKC>
__global__ __launch_bounds__(WM * WN * WK * 64, WK > 1 ? 4 : 2) void gemm_f32_kernel(GemmDesc g) {
  constexpr int NT = WM * WN * WK * 64, KT = f32_kt(WK);
  constexpr int TM = BM / WM, TN = BN / WN, MI = TM / 32, NI = TN / 32, GRP = KT / 8 / WK;
  typedef Tile<BM, KT, AK, NT> TA;
  typedef Tile<BN, KT, BKC, NT> TB;
  extern __shared__ __attribute__((aligned(16))) float sm[];
  float* As = sm;                          // [2][TA::FLOATS]
  float* Bs = sm + 2 * TA::FLOATS;         // [2][TB::FLOATS]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wk = wave / (WM * WN), wmn = wave % (WM * WN), wm = wmn / WN, wn = wmn % WN;
  const int lr = lane & 31, lh = lane >> 5;
  const int ntn = (g.N + BN - 1) / BN;
  const int tile = xcd_range(blockIdx.x, gridDim.x);
  const int m0 = (tile / ntn) * BM, n0 = (tile % ntn) * BN;
  const float* A = (const float*)g.A;
  const float* B = (const float*)g.B;
  const int64_t lda = AK ? g.a_rs : g.a_cs, ldb = BKC ? g.b_cs : g.b_rs;
  f32x16 acc[MI][NI];
#pragma unroll
  for (int mi = 0; mi < MI; ++mi)
#pragma unroll
    for (int ni = 0; ni < NI; ++ni)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[mi][ni][r] = 0.f;
  // column sums of B (the bias gradient of the layer): the first row of tiles adds up what passes through LDS
  constexpr int SG = NT / BN;                              // threads per column
  const bool do_bsum = !BKC && g.bsum && m0 == 0;          // uniform over the workgroup
  float csum = 0.f;
  // k-tile kt is multiplied from LDS while kt + 1 goes from registers to the other buffer and kt + 2, kt + 3 are on
  // their way from memory in two register stages
  TA ta[2];
  TB tb[2];
  const int nk = (g.K + KT - 1) / KT;
  auto fetch = [&](int st, int kt) __attribute__((always_inline)) {
    ta[st].fetch(A, lda, m0, g.M, kt * KT, g.K, tid);
    tb[st].fetch(B, ldb, n0, g.N, kt * KT, g.K, tid);
  };
  auto stash = [&](int st, int buf) __attribute__((always_inline)) {
    ta[st].stash(As + buf * TA::FLOATS, tid);
    tb[st].stash(Bs + buf * TB::FLOATS, tid);
  };
  auto step = [&](int par, int kt) __attribute__((always_inline)) {        // par = kt & 1, a constant
    if (kt + 1 < nk) stash(par ^ 1, par ^ 1);
    if (kt + 3 < nk) fetch(par ^ 1, kt + 3);
    const float* a = As + par * TA::FLOATS;
    const float* b = Bs + par * TB::FLOATS;
#pragma unroll
    for (int q = 0; q < GRP; ++q) {
      const int grp = q * WK + wk;
      f32x4 fa[MI], fb[NI];
#pragma unroll
      for (int mi = 0; mi < MI; ++mi) fa[mi] = TA::frag(a, wm * TM + mi * 32 + lr, grp, lh);
#pragma unroll
      for (int ni = 0; ni < NI; ++ni) fb[ni] = TB::frag(b, wn * TN + ni * 32 + lr, grp, lh);
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
          for (int ni = 0; ni < NI; ++ni)
            acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[mi][j], fb[ni][j], acc[mi][ni], 0, 0, 0);
    }
    if (do_bsum)
      for (int k = tid / BN; k < KT; k += SG) csum += b[k * TB::LD + tid % BN];
    __syncthreads();
  };
  fetch(0, 0);
  if (nk > 1) fetch(1, 1);
  stash(0, 0);
  if (nk > 2) fetch(0, 2);
  __syncthreads();
  for (int kt = 0; kt < nk; kt += 2) {
    step(0, kt);
    if (kt + 1 < nk) step(1, kt + 1);
  }
  if (do_bsum) {
    sm[tid] = csum;
    __syncthreads();
    if (tid < BN && n0 + tid < g.N) {
      float s = sm[tid];
#pragma unroll
      for (int i = 1; i < SG; ++i) s += sm[i * BN + tid];
      g.bsum[n0 + tid] = s;
    }
    __syncthreads();
  }
  // Epilogue.  Every wavefront puts its sums into LDS (element r of a 32 x 32 accumulator: row 8 (r / 4) + 4 h + r % 4,
  // column lane % 32), then the whole workgroup walks the tile in pieces of four columns, adding the copies of the
  // wavefronts that shared the k-tiles in order.  One loop, so that the code is short: written out per accumulator
  // element (erff and expf 16 to 64 times over) the kernels were 22 - 89 KB of code, fetched anew by every launch.
  constexpr int LDP = BN + 4;
#pragma unroll
  for (int mi = 0; mi < MI; ++mi)
#pragma unroll
    for (int ni = 0; ni < NI; ++ni)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        sm[(wk * BM + wm * TM + mi * 32 + 8 * (r >> 2) + 4 * lh + (r & 3)) * LDP + wn * TN + ni * 32 + lr] = acc[mi][ni][r];
  __syncthreads();
  float* C = (float*)g.C;
#pragma unroll 1
  for (int it = tid; it < BM * BN / 4; it += NT) {
    const int lrow = it / (BN / 4), lcol = it % (BN / 4) * 4, m = m0 + lrow, n = n0 + lcol;
    if (m >= g.M || n >= g.N) continue;
    f32x4 v = *(const f32x4*)(sm + lrow * LDP + lcol);
#pragma unroll
    for (int w = 1; w < WK; ++w) v += *(const f32x4*)(sm + (w * BM + lrow) * LDP + lcol);
    if (g.bias) v += *(const f32x4*)(g.bias + n);
    int64_t row = m;
    if (g.remap_np > 0) {
      row = (int64_t)m + m / g.remap_np + 1;
      v += *(const f32x4*)(g.pos + (int64_t)(m % g.remap_np + 1) * g.N + n);
    }
    const int64_t off = row * g.ldc + n;
    if (g.act == ACT_GELU) {
      if (g.aux) *(f32x4*)((float*)g.aux + off) = v;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = gelu_f(v[e]);
    } else if (g.act == ACT_GELU_BWD) {
      const f32x4 u = *(const f32x4*)((const float*)g.aux + off);
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] *= gelu_grad_f(u[e]);
    }
    if (g.res) v += *(const f32x4*)((const float*)g.res + (g.ldr ? row * g.ldr + n : off));
    *(f32x4*)(C + off) = v;
  }
}

template <int BM, int BN, int WM, int WN, int WK, bool AK, bool BKC>
void launch(const GemmDesc& g, hipStream_t s) {
  constexpr int NT = WM * WN * WK * 64, KT = f32_kt(WK);
  constexpr size_t tiles_f = 2 * (size_t)(Tile<BM, KT, AK, NT>::FLOATS + Tile<BN, KT, BKC, NT>::FLOATS);
  constexpr size_t sums_f = (size_t)WK * BM * (BN + 4);
  constexpr size_t lds = sizeof(float) * (tiles_f > sums_f ? tiles_f : sums_f);
  auto kern = gemm_f32_kernel<BM, BN, WM, WN, WK, AK, BKC>;
  static bool attr_set = false;
  if (!attr_set) {
    (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    attr_set = true;
  }
  const int tiles = ((g.M + BM - 1) / BM) * ((g.N + BN - 1) / BN);
  kern<<<tiles, NT, lds, s>>>(g);
}

// Which block tile: the one with the least matrix time on the busiest CU, ceil(tiles / 256) x tile area x K, the
// smaller tiles priced up by what their operand traffic and their sums over wavefronts cost.  The prices are set by hand, not
// fitted.  Steps with every product forced to 128, 64 and 32, and by this rule, in us: DeiT-S, a third of the tokens gone at
// three places, 1 image 4919, 1815, 1059, 1058; 8 images 5896, 2248, 1772, 1760; 32 images 9727, 4757, 4642, 4417; 8 images
// with all tokens 9773, 3852, 3378, 3530; one 192-wide block, 2 sequences of 65 442, 186, 130, 130.
int f32_pick(const GemmDesc& g) {
  const int edge[3] = {128, 64, 32};
  const float price[3] = {1.0f, 1.15f, 1.6f};
  int best = 0;
  float least = 0.f;
  for (int i = 0; i < 3; ++i) {
    const int64_t tiles = (int64_t)((g.M + edge[i] - 1) / edge[i]) * ((g.N + edge[i] - 1) / edge[i]);
    const float t = (float)((tiles + 255) / 256) * edge[i] * edge[i] * price[i];
    if (i == 0 || t < least) { best = i; least = t; }
  }
  return best;
}

template <bool AK, bool BKC>
void launch_form(const GemmDesc& g, hipStream_t s) {
  switch (f32_pick(g)) {
    case 0: launch<128, 128, 2, 2, 1, AK, BKC>(g, s); break;
    case 1: launch<64, 64, 2, 2, 2, AK, BKC>(g, s); break;
    default: launch<32, 32, 1, 1, 8, AK, BKC>(g, s); break;
  }
}

}  // namespace

// fp32 operands in one of the three forms a linear layer has, vectors of four along the contiguous index
bool gemm_f32_supported(const GemmDesc& g) {
  if (!g.in_f32 || !g.out_f32 || g.grp_off || g.ln_colsum || g.M < 1 || g.N < 4 || g.K < 1) return false;
  const bool ak = g.a_cs == 1, am = g.a_rs == 1 && !ak, bk = g.b_rs == 1, bn = g.b_cs == 1 && !bk;
  if (!((ak && (bn || bk)) || (am && bn))) return false;
  if (ak && (g.K % 4 || g.a_rs % 4)) return false;
  if (am && (g.M % 4 || g.a_cs % 4)) return false;
  if (bk && (g.K % 4 || g.b_cs % 4)) return false;
  if (bn && (g.N % 4 || g.b_rs % 4)) return false;
  if (g.N % 4 || g.ldc % 4 || g.ldr % 4) return false;
  const uintptr_t all = (uintptr_t)g.A | (uintptr_t)g.B | (uintptr_t)g.C | (uintptr_t)g.bias | (uintptr_t)g.aux | (uintptr_t)g.res |
                        (uintptr_t)g.pos;
  return (all & 15) == 0 && (!g.bsum || bn);
}

void gemm_f32(const GemmDesc& g, hipStream_t s) {
  if (g.a_cs != 1) launch_form<false, false>(g, s);          // weight gradient
  else if (g.b_rs == 1) launch_form<true, true>(g, s);       // input gradient
  else launch_form<true, false>(g, s);                       // forward
}

}  // namespace bsr
