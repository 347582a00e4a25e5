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
// Measured, chains of launches, operands staged through registers -> straight into LDS: 1576 x 384 x 1536 42.4 -> 30.5 us,
// 536 x 384 x 1536 16.9 -> 12.8, 1576 x 1536 x 384 30.6 -> 28.6 (65 TFLOP/s; the matrix cores alone 23).
//
// The contraction index of an MFMA is a dummy: MFMA j of a group of 8 uses k = 4 h + j for wave half h, so a lane's
// four operands of four MFMAs are four consecutive floats.  An operand whose k is contiguous in memory is read with one
// 16-byte LDS read per four MFMAs; an operand whose row index is contiguous lies as [k][row] and is read with four 4-byte
// reads.
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

// Loads that go straight into LDS: lane l of a wavefront writes 16 bytes at the wavefront's LDS address + 16 l
#define BSR_GLOBAL_PTR(p) ((const void __attribute__((address_space(1)))*)(p))
#define BSR_LDS_VOID(p) ((void __attribute__((address_space(3)))*)(p))
__device__ __forceinline__ void wait_vmcnt0() { __builtin_amdgcn_s_waitcnt((0x7 << 4) | (0xF << 8)); }
__device__ __forceinline__ void wait_lgkmcnt0() { __builtin_amdgcn_s_waitcnt(0xF | (0x3 << 14) | (0x7 << 4)); }

// k-tile: long where the wavefronts share it, since a tile that is alone on its CU is done with 32 k long before the
// next loads return (64 x 64 tiles at M = 1576, K = 384: 30 us with k-tiles of 32 fetched one ahead)
__host__ __device__ constexpr int f32_kt(int wk) { return wk == 1 ? 32 : wk == 2 ? 64 : 128; }

// One operand's tile in LDS: R rows (of the output index) x KT; KC: k contiguous in memory.  KC tiles lie as panels of 32 k,
// rows of eight 16-byte chunks, chunk c of row r at position c ^ swz(r) (16 rows that read the same chunk then hit every bank
// once; the permutation is applied to the global address a lane loads from); the others lie as [k][row].
__device__ inline int swz(int row) { return (row & 7) ^ ((row >> 3) & 1); }
template <int R, int KT, bool KC, int NT>
struct Tile {
  static constexpr int FLOATS = R * KT;
  static constexpr int NCH = R * KT / 4 / NT;                    // load instructions per thread
  static_assert(R * KT / 4 % NT == 0 && NCH >= 1, "every thread carries whole chunks");
  // output row (or first of four) and k of the chunk that thread tid's load i brings, relative to the tile
  __device__ static __forceinline__ void where(int tid, int i, int& r, int& k) {
    const int c = tid + NT * i;
    if (KC) { r = c / 8 % R; k = c / (8 * R) * 32 + (c % 8 ^ swz(r)) * 4; }
    else { r = c % (R / 4) * 4; k = c / (R / 4); }
  }
  // p: operand, ld: floats between memory rows, r0: first output row of the tile, rows / K: extents.  Rows past the end
  // repeat valid ones (never stored), k past the end too (cleared below).
  __device__ static __forceinline__ void load(float* s, const float* __restrict__ p, int64_t ld, int r0, int rows, int k0, int K, int tid) {
    float* dst = s + __builtin_amdgcn_readfirstlane(tid >> 6) * 256;
    const bool whole = k0 + KT <= K;
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      int r, k;
      where(tid, i, r, k);
      r += r0;
      k += k0;
      if (!whole) k = min(k, K - (KC ? 4 : 1));
      __builtin_amdgcn_global_load_lds(BSR_GLOBAL_PTR(KC ? p + (int64_t)min(r, rows - 1) * ld + k : p + (int64_t)k * ld + min(r, rows - 4)),
                                       BSR_LDS_VOID(dst + NT * 4 * i), 16, 0, 0);
    }
  }
  // what this thread has loaded of k >= K becomes zero
  __device__ static __forceinline__ void clear(float* s, int k0, int K, int tid) {
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      int r, k;
      where(tid, i, r, k);
      if (k0 + k >= K) *(f32x4*)(s + (tid + NT * i) * 4) = f32x4{0.f, 0.f, 0.f, 0.f};
    }
  }
  // four consecutive k of output row r: k-group grp of 8, wave half h
  __device__ static __forceinline__ f32x4 frag(const float* s, int r, int grp, int h) {
    if constexpr (KC) {
      const int chunk = grp * 2 + h;
      return *(const f32x4*)(s + (chunk / 8 * R + r) * 32 + (chunk % 8 ^ swz(r)) * 4);
    } else {
      f32x4 f;
#pragma unroll
      for (int j = 0; j < 4; ++j) f[j] = s[(grp * 8 + h * 4 + j) * R + r];
      return f;
    }
  }
};

// Operand tiles go straight into two stages in LDS, one k-tile ahead, one barrier per k-tile.  (Staged through
// registers, the branches around the last k-tiles made the compiler wait for every load in flight at each LDS write: loads
// and matrix work took turns, 23 + 25 us of the 42 us of 1576 x 384 x 1536.  A ring with its depth as a parameter, always two: fp32 steps
// of 1 .. 8 images of DeiT-S and of the 192-wide block took 2 % longer, DeiT-S of 8 images 1571 -> 1544 us.)
template <int BM, int BN, int WM, int WN, int WK, bool AK, bool BKC> struct F32Body {
  static constexpr int NT = WM * WN * WK * 64, KT = f32_kt(WK);
  typedef Tile<BM, KT, AK, NT> TA;
  typedef Tile<BN, KT, BKC, NT> TB;
  static constexpr int STAGE = TA::FLOATS + TB::FLOATS;
  static constexpr size_t LDS = sizeof(float) * (2 * (size_t)STAGE > (size_t)WK * BM * (BN + 4) ? 2 * (size_t)STAGE : (size_t)WK * BM * (BN + 4));
  static int tiles(const GemmDesc& g) { return ((g.M + BM - 1) / BM) * ((g.N + BN - 1) / BN); }
  // one tile; sizes and operands of g are the arguments
  __device__ static __forceinline__ void run(const float* A, const float* B, int64_t lda, int64_t ldb, GemmDesc& g, int tile);
};
template <int BM, int BN, int WM, int WN, int WK, bool AK, bool BKC>
__device__ __forceinline__ void F32Body<BM, BN, WM, WN, WK, AK, BKC>::run(const float* A, const float* B, int64_t lda, int64_t ldb, GemmDesc& g,
                                                                         int tile) {
  constexpr int TM = BM / WM, TN = BN / WN, MI = TM / 32, NI = TN / 32, GRP = KT / 8 / WK;
  extern __shared__ __attribute__((aligned(16))) float sm[];      // [2][STAGE]: A rows, then B rows
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wk = wave / (WM * WN), wmn = wave % (WM * WN), wm = wmn / WN, wn = wmn % WN;
  const int lr = lane & 31, lh = lane >> 5;
  const int ntn = (g.N + BN - 1) / BN;
  const int m0 = (tile / ntn) * BM, n0 = (tile % ntn) * BN;
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
  const int nk = (g.K + KT - 1) / KT;
  auto issue = [&](int kt, int st) __attribute__((always_inline)) {
    TA::load(sm + st * STAGE, A, lda, m0, g.M, kt * KT, g.K, tid);
    TB::load(sm + st * STAGE + TA::FLOATS, B, ldb, n0, g.N, kt * KT, g.K, tid);
  };
  issue(0, 0);
  for (int kt = 0; kt < nk; ++kt) {
    const int st = kt & 1;
    wait_vmcnt0();
    float* a = sm + st * STAGE;
    float* b = a + TA::FLOATS;
    if ((kt + 1) * KT > g.K) {
      TA::clear(a, kt * KT, g.K, tid);
      TB::clear(b, kt * KT, g.K, tid);
    }
    wait_lgkmcnt0();                                       // this wavefront has read k-tile kt - 1
    __builtin_amdgcn_s_barrier();
    if (kt + 1 < nk) issue(kt + 1, st ^ 1);
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
      for (int k = tid / BN; k < KT; k += SG) csum += b[k * BN + tid % BN];
  }
  __syncthreads();
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
__global__ __launch_bounds__(WM * WN * WK * 64, WK > 1 ? 4 : 2)
void gemm_f32_kernel(const float* A, const float* B, int64_t lda, int64_t ldb, int M, int N, int K, int tiles, GemmDesc g) {
  g.M = M; g.N = N; g.K = K;               // (in front of the description: these arrive in registers with the wavefront)
  F32Body<BM, BN, WM, WN, WK, AK, BKC>::run(A, B, lda, ldb, g, xcd_range(blockIdx.x, tiles));
}

template <int BM, int BN, int WM, int WN, int WK, bool AK, bool BKC>
void launch(const GemmDesc& g, hipStream_t s) {
  using Body = F32Body<BM, BN, WM, WN, WK, AK, BKC>;
  auto kern = gemm_f32_kernel<BM, BN, WM, WN, WK, AK, BKC>;
  static bool attr_set = false;
  if (!attr_set) {
    (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)Body::LDS);
    attr_set = true;
  }
  const int tiles = Body::tiles(g);
  kern<<<tiles, Body::NT, Body::LDS, s>>>((const float*)g.A, (const float*)g.B, AK ? g.a_rs : g.a_cs, BKC ? g.b_cs : g.b_rs, g.M, g.N, g.K, tiles, g);
}

// Both gradients of a layer in one launch: dx = dy W^T (dg) and dW = x^T dy (wg) read the same dy and neither reads what the other writes.
// The workgroups with the longer sums come first, the others fill the CUs they leave; tiles and sums are those of two launches, so the results
// are the same bits.  What it saves is a launch, and the CUs that few tiles leave idle (gemm_f32_pair below); steps
// of DeiT-S with 1, 4 and 8 images 850 -> 790, 1069 -> 996, 1445 -> 1402 us, of a 192-wide block with 2 sequences 110 -> 94.
// (The 14 dwords up to wg_blocks come in registers.)
template <class DG, class WG>
__global__ __launch_bounds__(512, 4) void gemm_f32_pair_kernel(const float* dy, const float* w, const float* x, int M, int in, int out, unsigned dy_rs,
                                                               unsigned w_rs, unsigned x_rs, int dg_blocks, int wg_blocks, GemmDesc dg, GemmDesc wg) {
  static_assert(DG::NT == 512 && WG::NT == 512, "");
  const bool wg_first = M >= out;
  const int first = wg_first ? wg_blocks : dg_blocks;
  const bool mine = (int)blockIdx.x < first;
  const int block = mine ? blockIdx.x : blockIdx.x - first;
  if (mine == wg_first) {
    wg.M = in; wg.N = out; wg.K = M;
    WG::run(x, dy, x_rs, dy_rs, wg, xcd_range(block, wg_blocks));
  } else {
    dg.M = M; dg.N = in; dg.K = out;
    DG::run(dy, w, dy_rs, w_rs, dg, xcd_range(block, dg_blocks));
  }
}
template <class DG, class WG> void launch_pair(const GemmDesc& dg, const GemmDesc& wg, hipStream_t s) {
  constexpr size_t lds = DG::LDS > WG::LDS ? DG::LDS : WG::LDS;
  auto kern = gemm_f32_pair_kernel<DG, WG>;
  static bool attr_set = false;
  if (!attr_set) {
    (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    attr_set = true;
  }
  const int nd = DG::tiles(dg), nw = WG::tiles(wg);
  kern<<<nd + nw, 512, lds, s>>>((const float*)dg.A, (const float*)dg.B, (const float*)wg.A, dg.M, dg.N, dg.K, (unsigned)dg.a_rs, (unsigned)dg.b_cs,
                                 (unsigned)wg.a_cs, nd, nw, dg, wg);
}

// Which block tile: the one that a model finishes first.  With t tiles, time = c0 + ceil(t / 256) (c1 + c2 K / 100) + t / 256
// (c3 + c4 K / 100) + ceil(t / 512) (c5 + c6 K / 100) microseconds (rounds of one workgroup per CU, work, rounds of two), fitted to chains
// of equal launches of the three forms (264 products: 65 .. 6304 rows, 192 and 384 wide).  Its picks take 0.1 % longer than the
// fastest tile; tile areas with prices set by hand 1.0 %, 32 x 32 always 3.9 %.  At other widths the model extrapolates.
// The fewer k of a tile a wavefront adds up, the closer a sum is to its value in 64 bits, so no product takes a larger tile than `most`, the
// least of tile area x rounds of the CUs with those prices (DeiT-S steps of 1 .. 8 images: weight gradients over a few dozen tokens).
int f32_pick(const GemmDesc& g) {
  const int edge[3] = {128, 64, 32};
  const float c[3][7] = {{6.180f, 0.000f, 5.645f, 3.077f, 0.964f, 1.018f, 0.500f},
                         {3.079f, 0.387f, 1.480f, 0.514f, 0.321f, 0.420f, 0.279f},
                         {2.598f, 0.505f, 0.421f, 0.453f, 0.032f, 0.137f, 0.152f}};
  const float price[3] = {1.0f, 1.15f, 1.6f};
  int64_t tiles[3];
  int most = 0, best = 0;
  float least = 0.f;
  for (int i = 0; i < 3; ++i) {
    tiles[i] = (int64_t)((g.M + edge[i] - 1) / edge[i]) * ((g.N + edge[i] - 1) / edge[i]);
    const float area = (float)((tiles[i] + 255) / 256) * edge[i] * edge[i] * price[i];
    if (i == 0 || area < least) { most = i; least = area; }
  }
  const float k = 0.01f * g.K;
  for (int i = most; i < 3; ++i) {
    const float t = c[i][0] + (float)((tiles[i] + 255) / 256) * (c[i][1] + c[i][2] * k) + (float)tiles[i] / 256.f * (c[i][3] + c[i][4] * k) +
                    (float)((tiles[i] + 511) / 512) * (c[i][5] + c[i][6] * k);
    if (i == most || t < least) { best = i; least = t; }
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

// The two gradients of one layer.  One launch, unless a product takes the 128 x 128 tiles, which have half the wavefronts: it was the faster
// one wherever it was measured.  Steps of one block, two launches -> one (GPU time): 64 wide, 130 .. 4160 rows 0.84 .. 0.92 times as long, 128 wide, 394 .. 6304
// rows 0.85 .. 0.89, 192 wide, 65 .. 6304 rows 0.83 .. 0.91 (16 sequences of 65 tokens 142 -> 129 us, 32 209 -> 183), 256 wide, 197 .. 3152 rows 0.88 .. 0.94,
// 384 wide, 197 .. 6304 rows 0.87 .. 0.95, 768 wide, 197 .. 1576 rows 0.90 .. 0.97.
void gemm_f32_pair(const GemmDesc& dg, const GemmDesc& wg, hipStream_t s) {
  const bool layer = dg.a_cs == 1 && dg.b_rs == 1 && wg.a_rs == 1 && wg.a_cs != 1 && wg.b_cs == 1 && dg.A == wg.B && dg.a_rs == wg.b_rs && dg.M == wg.K &&
                     dg.N == wg.M && dg.K == wg.N && std::max({dg.a_rs, dg.b_cs, wg.a_cs}) <= (int64_t)INT32_MAX;
  const int di = f32_pick(dg), wi = f32_pick(wg);
  if (!layer || di == 0 || wi == 0) {
    gemm_f32(dg, s);
    gemm_f32(wg, s);
    return;
  }
  typedef F32Body<64, 64, 2, 2, 2, true, true> D1;
  typedef F32Body<32, 32, 1, 1, 8, true, true> D2;
  typedef F32Body<64, 64, 2, 2, 2, false, false> W1;
  typedef F32Body<32, 32, 1, 1, 8, false, false> W2;
  if (di == 1) wi == 1 ? launch_pair<D1, W1>(dg, wg, s) : launch_pair<D1, W2>(dg, wg, s);
  else wi == 1 ? launch_pair<D2, W1>(dg, wg, s) : launch_pair<D2, W2>(dg, wg, s);
}

}  // namespace bsr
