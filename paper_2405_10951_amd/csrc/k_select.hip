// Token selection of a drop location (Sec. 4.1, Eq. 6) in one launch: head mean of the class token's softmax rows, the
// k best patch tokens, the rows handed on (class token, kept tokens in ascending order, optionally one token fused
// from the dropped ones) and the LayerNorm that follows them.
//
// What bounds it: launches (the rows are a few MB).  So every workgroup of an image finds the kept set by itself, which
// takes one wavefront about a microsecond, and goes on with its share of the rows; ranking, gather, fusion and
// LayerNorm took four launches (8 + 5 + 60 + 6 us at 27 images of 197 tokens, 768 wide).
// The kept set is found by bisection over the bits of the scores: steps fix, from the top down, one or two bits each of the largest
// value that at least k scores reach, each a compare and ballot per 64 scores and candidate, and stop once exactly k do (mostly half
// way down).  (Calls in a row, one bit a step to the last bit -> this: 128 images of 196 tokens, 768 wide, 13.3 -> 10.8 us, 32 of 576 14.3 -> 11.5,
// 4 of 1023 15.2 -> 11.4; in a step with its LayerNorm, 32 images of 196 tokens 10.8 -> 7.9.)  (Counting for every score how many beat it takes n^2 compares: 32 us at 576 tokens.)
#include <algorithm>

#include "rowops.h"

namespace bsr {

namespace {

constexpr int MAX_N = 1024, SEL_WAVES = 8;

// order-preserving key, larger is better; -0 and +0 are one value; a NaN (a diverged step) ranks last with -infinity,
// so that the order stays total and exactly k tokens are kept.  Never 0.
__device__ inline unsigned score_key(float v) {
  v = v == v ? v + 0.0f : -INFINITY;
  const unsigned u = __float_as_uint(v);
  return (u & 0x80000000u) ? ~u : u | 0x80000000u;
}

// One wavefront: ascending indices of the k best of sc[0 .. n) into list, equal scores to the lower index.  n <= 64 NC; BITS are fixed
// per step (with 16 chunks of scores three counts a step take longer than two steps).
template <int NC, int BITS>
__device__ __forceinline__ void select_wave(const float* sc, int n, int k, int lane, int32_t* list) {
  unsigned key[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) key[c] = c * WAVE + lane < n ? score_key(sc[c * WAVE + lane]) : 0u;
  auto count = [&](auto better) __attribute__((always_inline)) {
    int cnt = 0;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      if (NC > 4 && c * WAVE >= n) break;
      cnt += __popcll(__ballot(better(key[c])));
    }
    return cnt;
  };
  unsigned kth = 0;                         // in the end the k-th largest key, or a value that exactly the k best reach
#pragma unroll 1
  for (int bit = 32 - BITS; bit >= 0; bit -= BITS) {
    constexpr int ND = (1 << BITS) - 1;
    int reach[ND], d = 0, at = 0;           // scores that reach digit 1, 2, ..; the largest digit that k reach, and how many do
#pragma unroll
    for (int i = 0; i < ND; ++i) {
      const unsigned cand = kth | ((unsigned)(i + 1) << bit);
      reach[i] = count([&](unsigned x) { return x >= cand; });
    }
#pragma unroll
    for (int i = 0; i < ND; ++i)
      if (reach[i] >= k) { d = i + 1; at = reach[i]; }
    kth |= (unsigned)d << bit;
    if (d && at == k) break;
  }
  int ties = k - count([&](unsigned x) { return x > kth; });      // of the equal ones, the first so many
  int base = 0;
  const unsigned long long below = (1ull << lane) - 1ull;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    if (NC > 4 && c * WAVE >= n) break;
    const bool eq = key[c] == kth;
    const unsigned long long em = __ballot(eq);
    const bool keep = key[c] > kth || (eq && __popcll(em & below) < ties);
    ties -= min(ties, (int)__popcll(em));
    const unsigned long long km = __ballot(keep);
    if (keep) list[base + __popcll(km & below)] = c * WAVE + lane;
    base += __popcll(km);
  }
}

// Workgroup (image b, part y): y < row_parts hands on rows y * rows .. of [class; kept]; y == row_parts (only with
// a.fw) makes the fused token.  MAXC == 0: rows are copied only; otherwise LayerNorm follows.  Held to the registers of four workgroups
// a CU, which launch() counts on (at three, 16 images of 576 tokens took a second round: 12 -> 18 us).
template <typename T, int MAXC>
__global__ __launch_bounds__(SEL_WAVES * WAVE, MAXC <= 2 ? 8 : 1) void select_kernel(SelectArgs a, int rows, int row_parts) {
  constexpr int V = Chunk<T>::V, MC = MAXC ? MAXC : 1;
  typedef typename Chunk<T>::vec vec;
  __shared__ float sc[MAX_N];
  __shared__ int32_t list[MAX_N];
  __shared__ float fused[SEL_WAVES * V * WAVE];
  const int b = blockIdx.x, part = blockIdx.y, tid = threadIdx.x, lane = tid % WAVE, n = a.T - 1, k = a.k;
  const int wave = __builtin_amdgcn_readfirstlane(tid / WAVE);
  const bool first = part == 0;
  if (a.cls_prob) {                         // heads in ascending order, then divided by H
    for (int j = tid; j < n; j += SEL_WAVES * WAVE) {
      const float* p = a.cls_prob + (int64_t)b * a.H * a.T + 1 + j;
      float v = 0.f;
      for (int h0 = 0; h0 < a.H; h0 += 12) {            // (twelve loads at a time)
        float t[12];
#pragma unroll
        for (int u = 0; u < 12; ++u) t[u] = p[(int64_t)min(h0 + u, a.H - 1) * a.T];
#pragma unroll
        for (int u = 0; u < 12; ++u)
          if (h0 + u < a.H) v += t[u];
      }
      v /= (float)a.H;
      sc[j] = v;
      if (first && a.scores) a.scores[(int64_t)b * n + j] = v;
    }
  } else if (!a.forced) {
    for (int j = tid; j < n; j += SEL_WAVES * WAVE) sc[j] = a.scores[(int64_t)b * n + j];
  }
  if (a.forced)
    for (int i = tid; i < k; i += SEL_WAVES * WAVE) list[i] = a.forced[(int64_t)b * k + i];
  __syncthreads();
  if (!a.forced) {
    if (wave == 0) {
      if (n <= 4 * WAVE) select_wave<4, 2>(sc, n, k, lane, list);
      else select_wave<MAX_N / WAVE, 1>(sc, n, k, lane, list);
    }
    __syncthreads();
  }
  if (first)
    for (int i = tid; i < k; i += SEL_WAVES * WAVE) {
      if (a.idx) a.idx[(int64_t)b * k + i] = list[i];
      if (a.idx2) a.idx2[(int64_t)b * k + i] = list[i];
    }
  if (!a.x) return;
  const int D = a.D, nch = D / V, T_out = k + 1 + (a.fw ? 1 : 0);
  const T* xb = (const T*)a.x + (int64_t)b * a.T * D;
  const int64_t out0 = (int64_t)b * T_out;
  auto layernorm = [&](const float (&v)[MC][V], int64_t m) __attribute__((always_inline)) {
    if constexpr (MAXC > 0) {
      RowParams<T, MAXC, MAXC == 1> par;
      par.ahead(a.gamma, a.beta, nch, lane);
      layernorm_row(v, par, D, lane, a.gamma, a.beta, a.eps, (T*)a.y + m * D, a.mean ? a.mean + m : nullptr,
                             a.rstd ? a.rstd + m : nullptr);
    }
  };
  if (part < row_parts) {
    const int end = min((part + 1) * rows, k + 1);
    for (int i = part * rows + wave; i < end; i += SEL_WAVES) {
      const T* src = xb + (int64_t)(i == 0 ? 0 : 1 + list[i - 1]) * D;
      const int64_t m = out0 + i;
      T* dst = (T*)a.x_kept + m * D;
      if constexpr (MAXC == 0) {
        for (int c = lane; c < nch; c += WAVE) *(vec*)(dst + c * V) = *(const vec*)(src + c * V);
      } else {
        float v[MC][V];
        vec raw[MC];
        load_row<T, MC>(src, nch, lane, raw, v);
#pragma unroll
        for (int q = 0; q < MC; ++q)
          if (lane + q * WAVE < nch) *(vec*)(dst + (lane + q * WAVE) * V) = raw[q];
        layernorm(v, m);
      }
    }
    return;
  }
  // The fused token: sum over the dropped j of w_j x[1+j], w_j = a_j / sum of the dropped a_j, as row k+1.  fw receives
  // the weights (0 for kept tokens), the backward pass reuses them as constants.
  for (int i = tid; i < k; i += SEL_WAVES * WAVE) sc[list[i]] = 0.f;
  __syncthreads();
  float s = 0.f;                            // every wavefront adds all of them: the same order everywhere
  for (int j = lane; j < n; j += WAVE) s += sc[j];
  const float inv = 1.0f / wave_sum(s);
  for (int j = tid; j < n; j += SEL_WAVES * WAVE) a.fw[(int64_t)b * n + j] = sc[j] * inv;
  const int64_t m = out0 + k + 1;
  float v[MC][V] = {};
  // 64 chunks of the row at a time: every wavefront adds its share of the tokens, wavefront 0 the eight shares
  auto chunks = [&](int q, float (&o)[V]) __attribute__((always_inline)) {
    const int c = q * WAVE + lane;
    float acc[V];
#pragma unroll
    for (int e = 0; e < V; ++e) acc[e] = 0.f;
    if (c < nch) {
#pragma unroll 4
      for (int j = wave; j < n; j += SEL_WAVES) {
        const float w = sc[j] * inv;
        if (w == 0.f) continue;
        const vec t = *(const vec*)(xb + (int64_t)(1 + j) * D + c * V);
#pragma unroll
        for (int e = 0; e < V; ++e) acc[e] = fmaf(w, (float)t[e], acc[e]);
      }
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < V; ++e) fused[(wave * V + e) * WAVE + lane] = acc[e];
    __syncthreads();
    if (wave != 0 || c >= nch) return;
    vec t;
#pragma unroll
    for (int e = 0; e < V; ++e) {
      float f = acc[e];
#pragma unroll
      for (int w = 1; w < SEL_WAVES; ++w) f += fused[(w * V + e) * WAVE + lane];
      t[e] = (T)f;
      o[e] = (float)t[e];                   // LayerNorm sees the stored row
    }
    *(vec*)((T*)a.x_kept + m * D + c * V) = t;
  };
  if constexpr (MAXC == 0) {
    for (int q = 0; q * WAVE < nch; ++q) chunks(q, v[0]);
  } else {
#pragma unroll
    for (int q = 0; q < MC; ++q) chunks(q, v[q]);
    if (wave == 0) layernorm(v, m);
  }
}

template <typename T>
void launch(const SelectArgs& a, int B, bool with_ln, hipStream_t s) {
  // rows per workgroup: 8 (one per wavefront) for few images, up to 64 where the images alone fill the chip
  int rows = SEL_WAVES;
  while (rows < 64 && (int64_t)B * ((a.k + rows) / rows) > 1024) rows *= 2;
  const int row_parts = a.x ? (a.k + rows) / rows : 1;
  const dim3 grid(B, row_parts + (a.x && a.fw ? 1 : 0));
  if (with_ln)
    with_row_chunks<T>(a.D, [&](auto C) { select_kernel<T, decltype(C)::value><<<grid, SEL_WAVES * WAVE, 0, s>>>(a, rows, row_parts); });
  else
    select_kernel<T, 0><<<grid, SEL_WAVES * WAVE, 0, s>>>(a, rows, row_parts);
}

}  // namespace

// D: a multiple of 8.  Returns whether the LayerNorm asked for (a.y) was done: rows longer than ROW_MAX need their own.
bool select_tokens(const SelectArgs& a, int B, bool f32, hipStream_t s) {
  const bool with_ln = a.x && a.y && a.D <= ROW_MAX;
  if (B > 0) {
    if (f32) launch<float>(a, B, with_ln, s);
    else launch<bf16>(a, B, with_ln, s);
  }
  return with_ln;
}

}  // namespace bsr
