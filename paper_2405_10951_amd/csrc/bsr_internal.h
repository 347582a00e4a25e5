// Internal declarations shared by the translation units of libbsr_hip: kernel launchers take raw
// device pointers and a stream, never allocate and never synchronise.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace bsr {

typedef __bf16 bf16;

enum Act { ACT_NONE = 0, ACT_GELU = 1, ACT_GELU_BWD = 2 };

// C(m,n) = epilogue( sum_k A(m,k) * B(k,n) ), operands addressed through element strides so that
// one description covers X.W (forward), dY.W^T (Eq. 2) and X^T.dY (Eq. 4).
struct GemmDesc {
  const void* A = nullptr; int64_t a_rs = 0, a_cs = 0;   // A(m,k) = A[m*a_rs + k*a_cs]
  const void* B = nullptr; int64_t b_rs = 0, b_cs = 0;   // B(k,n) = B[k*b_rs + n*b_cs]
  void* C = nullptr;       int64_t ldc = 0;              // C(m,n) = C[row(m)*ldc + n]
  int M = 0, N = 0, K = 0;
  bool in_f32 = false;                                   // A and B are fp32 (else bf16)
  bool out_f32 = false;                                  // C is fp32 (else bf16)
  const float* bias = nullptr;                           // [N], added before the activation
  int act = ACT_NONE;
  void* aux = nullptr;       // ACT_GELU: if set, receives the pre-activation u (dtype of C, ld = ldc)
                             // ACT_GELU_BWD: the stored u; C = acc * GELU'(u)
  const void* res = nullptr; // residual added last (dtype of C, same row mapping)
  int64_t ldr = 0;           // its row stride; 0: ldc
  int remap_np = 0;          // > 0 (patch embedding): row(m) = m + m / np + 1, and pos[(m % np + 1), n]
  const float* pos = nullptr;//   is added; rows of CLS tokens are left untouched
  float* bsum = nullptr;     // weight-gradient form only (A^T and B share the token index k): if set,
                             //   receives sum_k B(k,n), the bias gradient of the same layer
  // Grouped form (expert FFNs over routed tokens): the token rows are cut into `groups` consecutive
  // ranges, range e = [grp_off[e], grp_off[e+1]) (device array), each with its own weight matrix.
  //   forward / dgrad: rows of A and C in range e use B + e*b_gs and bias + e*bias_gs
  //   wgrad:           the contraction runs over range e only and fills C + e*c_gs, bsum + e*bsum_gs
  const int32_t* grp_off = nullptr;
  int groups = 0;
  int64_t b_gs = 0, bias_gs = 0, c_gs = 0, bsum_gs = 0;
  // LayerNorm folded into the linear layer that follows it (frozen weights; NT form, K a multiple of 64):
  //   LN(x) W^T + b = rstd (x W'^T - mean colsum(W')) + b',   W' = W diag(gamma),  b' = b + W beta.
  // With ln_colsum set ([N], sum_k W'(n,k)), A is the raw x, B is W', bias is b'; the kernel takes mean and
  // 1/std of every row of A from the tiles it streams anyway and applies the formula in its epilogue.
  const float* ln_colsum = nullptr;
  float ln_eps = 0.f;
};

// ---- generic (any shape, fp32 or bf16 storage, fp32 arithmetic) ---------------------------------
void gemm_generic(const GemmDesc& g, hipStream_t s);
void attn_fwd_generic(const void* qkv, int B, int T, int H, int d, bool f32, void* out, float* lse,
                      float* cls_prob, hipStream_t s);
void attn_bwd_generic(const void* qkv, const void* out, const void* dout, const float* lse, int B,
                      int T, int H, int d, bool f32, float* delta, void* dqkv, hipStream_t s);

// ---- fp32 MFMA paths (any row count; contiguous extents in multiples of four, head size 64) -------
bool gemm_f32_supported(const GemmDesc& g);
void gemm_f32(const GemmDesc& g, hipStream_t s);
// input gradient and weight gradient of one layer (both supported), in one launch where their tiles allow it
void gemm_f32_pair(const GemmDesc& dg, const GemmDesc& wg, hipStream_t s);
bool attn_f32_supported(int T, int d);
void attn_fwd_f32(const float* qkv, int B, int T, int H, float* out, float* lse, float* cls_prob, hipStream_t s);
void attn_bwd_f32(const float* qkv, const float* out, const float* dout, const float* lse, int B, int T, int H,
                  float* dqkv, hipStream_t s);

// W'(n,k) = bf16(w[k,n] gamma[k]) as [out][in], colsum[n] = sum_k W'(n,k), bias_out[n] = bias[n] + sum_k beta[k] w[k,n]
// (w is the fp32 master matrix [in][out]; in a multiple of 8)
void ln_fold_weights(const float* w, const float* bias, const float* gamma, const float* beta, int in, int out,
                     bf16* w_t, float* colsum, float* bias_out, hipStream_t s);

// ---- bf16 MFMA paths --------------------------------------------------------------------------
bool gemm_mfma_supported(const GemmDesc& g);
// splitk_ws: fp32 scratch for the partial sums of split-K weight gradients (may be null: no split)
// A weight gradient whose tokens several workgroups share leaves fp32 partials that one more pass has to add up.  With a chain, that
// pass does not get a launch of its own: it rides on the NEXT weight-gradient launch
// (which works on the other half of the workspace), and the last one goes out with the sums of the LayerNorms (gemm_tn_take,
// ln_deferred_finish).  The sums and their order are the same either way.
struct TnReduce {
  const float* partial = nullptr;   // [splits][n]
  int64_t n = 0;
  int splits = 0;                   // partials
  float* out = nullptr;
  const float* bpartial = nullptr;  // [splits][nb] column sums (bias gradient), may be null
  int nb = 0;
  float* bout = nullptr;
};
// four elements of a sum of partials (or, past the matrix, up to four of the column sums): added in
// ascending order
__device__ inline void splitk_reduce_item(const TnReduce& r, int64_t item) {
  const int64_t i = item * 4;
  if (i >= r.n) {
    for (int64_t j = i - r.n; j < min(i - r.n + 4, (int64_t)r.nb); ++j) {
      float s = r.bpartial[j];
      for (int z = 1; z < r.splits; ++z) s += r.bpartial[(int64_t)z * r.nb + j];
      r.bout[j] = s;
    }
    return;
  }
  float4 s = *(const float4*)(r.partial + i);
  for (int z = 1; z < r.splits; ++z) {
    const float4 v = *(const float4*)(r.partial + (int64_t)z * r.n + i);
    s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
  }
  *(float4*)(r.out + i) = s;
}
__host__ __device__ inline int64_t splitk_reduce_items(const TnReduce& r) { return r.n / 4 + (r.nb + 3) / 4; }
struct TnChain {
  TnReduce pending;                 // pending.splits > 0: a reduction is waiting
  int slot = 0;                     // workspace half the next split launch writes
};
// tile: one of gemm_nt_tile_id() or what gemm_nt_runs_tile() gave, for the NT kernel (ignored by the others), 0 = the built-in model chooses
void gemm_mfma(const GemmDesc& g, float* splitk_ws, size_t splitk_ws_floats, hipStream_t s, int tile = 0,
               TnChain* chain = nullptr);
TnReduce gemm_tn_take(TnChain* chain);          // for a caller that adds the waiting partials up itself (splits 0: none wait)
// input gradient (NT) + weight gradient (TN) of one layer, in one launch when the NT tile shape has that form
void gemm_mfma_pair(const GemmDesc& nt, const GemmDesc& tn, float* splitk_ws, size_t splitk_ws_floats, hipStream_t s,
                    int tile = 0, TnChain* chain = nullptr);
// the block-tile shapes the NT kernel is instantiated for, and whether a GEMM is free to take any of them
int gemm_nt_tile_count();
constexpr int FEW_ROWS_ID = 9000000;           // + 1000 rows + columns: a tile of the kernel for products of few rows
constexpr int APART_ID = 10000000;             // + id of a shape that also names a layer's joint launch: its two launches, the input gradient in that shape
// id of the shape that really runs when `tile` is asked for (0: without a measured choice; wgrad: the weight gradient that goes out
// with g, or null; the workspace as in the call).  Asked for in turn, it runs the same.  FEW_ROWS_ID + ..: whatever is asked for
int gemm_nt_runs_tile(const GemmDesc& g, const GemmDesc* wgrad, size_t splitk_ws_floats, bool chained, int tile);
int gemm_nt_tile_id(int i);
// an id that the entry points take: 0, a shape above, or one that was a shape once (the model chooses in its place)
bool gemm_nt_tile_known(int id);
size_t gemm_nt_tile_lds_bytes(int id);          // dynamic LDS a workgroup of that shape holds
bool gemm_nt_tile_is_free(const GemmDesc& g);
size_t gemm_splitk_ws_floats(int dim, int mlp_hidden);

// Attention of query 0 (the class token) alone: out [B, H d], lse [B, H]; backward from a gradient at those rows, dqkv
// [B, T, 3 H d] written whole.  d: whole 16-byte pieces
bool attn_cls_supported(int T, int d, bool f32);
void attn_cls_fwd(const void* qkv, int B, int T, int H, int d, bool f32, void* out, float* lse, hipStream_t s);
void attn_cls_bwd(const void* qkv, const void* dout, const float* lse, int B, int T, int H, int d, bool f32,
                  void* dqkv, hipStream_t s);

bool attn_mfma_supported(int T, int d);
void attn_fwd_mfma(const void* qkv, int B, int T, int H, void* out, float* lse, float* cls_prob, hipStream_t s);
void attn_bwd_mfma(const void* qkv, const void* out, const void* dout, const float* lse, int B, int T, int H,
                   float* delta, void* dqkv, hipStream_t s);

// ---- row-wise / element-wise kernels ------------------------------------------------------------
void layernorm_fwd(const void* x, int64_t M, int D, const float* gamma, const float* beta, float eps,
                   bool f32, void* y, float* mean, float* rstd, hipStream_t s);
// res may be null, dx null to skip it.  res_period 0: a residual row per row; P > 0: rows 0, P, 2P, ... have one each
// (the residual then has M / P rows).
// idx: row m of dx is that of a token behind a drop (k + 1 rows per image, [class; kept], idx [B, k] ascending, distinct
// and below T - 1: nothing checks it, so lists of the selection only) and goes to its place among the T tokens before it; the dropped tokens' rows
// are set to zero
struct LnScatter { const int32_t* idx = nullptr; int k = 0, T = 0; };
template <typename T> struct LnRows { const T* x; const T* res; T* dx; int res_period; LnScatter sc; };
// dx = res + LN'(dy)
void layernorm_bwd_dx(const void* dy, const void* x, const float* mean, const float* rstd,
                      const float* gamma, const void* res, int64_t M, int D, bool f32, void* dx,
                      hipStream_t s, int res_period = 0, const LnScatter& sc = LnScatter());
// dgamma[j] = sum_m dy*xhat, dbeta[j] = sum_m dy ; partial is scratch of colsum_partial_floats()
void layernorm_bwd_params(const void* dy, const void* x, const float* mean, const float* rstd,
                          int64_t M, int D, bool f32, float* partial, float* dgamma, float* dbeta,
                          hipStream_t s);
// out[j] = sum_m a[m*ld + j]
void colsum(const void* a, int64_t M, int N, int64_t ld, bool f32, float* partial, float* out,
            hipStream_t s);
size_t colsum_partial_floats(int64_t M, int N);
// dx and the parameter gradients in one pass, with one final reduction for several layers: a call writes dx and its
// workgroup partials of dgamma / dbeta into `slot` (a buffer of its own of ln_deferred_partial_floats(D) floats, kept
// until the reduction) and adds an entry to the table; ln_deferred_finish adds the partials of every entry in one
// launch.  Shapes the one-pass kernel does not take, a null slot or a full table go through separate kernels.
constexpr int LN_DEFER_MAX = 32, LN_BWD_BLOCKS = 256;
struct LnDeferEntry { const float* partial; float* dgamma; float* dbeta; int blocks; };
struct LnDeferTable { LnDeferEntry e[LN_DEFER_MAX]; int count = 0; int D = 0; };
size_t ln_deferred_partial_floats(int D);
void layernorm_bwd(const void* dy, const void* x, const float* mean, const float* rstd, const float* gamma,
                   const void* res, int64_t M, int D, bool f32, void* dx, float* partial, float* slot, float* dgamma,
                   float* dbeta, LnDeferTable& t, hipStream_t s, int res_period = 0, const LnScatter& sc = LnScatter());
// whether rows of D can be scattered on the way out
bool layernorm_bwd_scatters(int D, bool f32);
// and the partials of the last weight gradient in the same launch (red.splits 0: none)
void ln_deferred_finish(LnDeferTable& t, const TnReduce& red, hipStream_t s);

// cls given: also writes the class-token rows x[b, 0, :] = cls + pos[0] of the token tensor x [B, T, D] (same launch
// on the 16-byte path)
void patchify(const void* img, int B, int C, int S, int P, bool f32, void* out, hipStream_t s,
              const float* cls = nullptr, const float* pos = nullptr, int T = 0, int D = 0, void* x = nullptr);
// bytes: a multiple of 16, both pointers aligned to 16 (a kernel of its own: the runtime's copy takes the host twice a launch)
void copy_rows(const void* src, void* dst, size_t bytes, hipStream_t s);
void write_cls_rows(const float* cls, const float* pos, int B, int T, int D, bool f32, void* x,
                    hipStream_t s);
// Token selection and what follows it, in one launch (k_select.hip).  Per image: scores = head mean of the class token's
// softmax rows (cls_prob [B,H,T], written to scores [B,T-1]) or, with cls_prob null, scores as given; the k best
// (forced [B,k]: these instead) go to idx and idx2, ascending; with x [B,T,D], rows [class; kept] go to x_kept
// (k + 1 rows per image; with fw one row more, the dropped tokens fused, and fw [B,T-1] receives the weights); with y also
// the LayerNorm of x_kept's rows.  Null pointers are skipped.
struct SelectArgs {
  const float* cls_prob = nullptr; int H = 0;
  float* scores = nullptr;
  const int32_t* forced = nullptr;
  int32_t *idx = nullptr, *idx2 = nullptr;
  int T = 0, k = 0, D = 0;
  const void* x = nullptr; void* x_kept = nullptr;
  float* fw = nullptr;
  const float *gamma = nullptr, *beta = nullptr; float eps = 0.f;
  void* y = nullptr; float *mean = nullptr, *rstd = nullptr;
};
bool select_tokens(const SelectArgs& a, int B, bool f32, hipStream_t s);    // true: the LayerNorm was done
// fw != null: dy has rows [CLS; kept; fused] and dropped tokens get fw times the fused token's gradient
void scatter_tokens(const void* dy, const int32_t* idx, int B, int T, int k, int D, bool f32,
                    void* dx, hipStream_t s, const float* fw = nullptr);
// Classification head, forward and backward, in two launches (class-token LayerNorm, logits, mean
// cross-entropy, and the gradients of the head, of the final LayerNorm and of the last block's output
// dx [B,Tl,D], whose non-class rows are set to zero).  xhat, z, dz: [B,D] fp32 scratch; logits, dlogits:
// [B,C] fp32; loss_rows [B].  head_takes: whether these kernels are the ones for a head (by size).
bool head_takes(int B, int D, int C, const float* w_head);
void head_fwd_bwd(const void* x, int B, int Tl, int D, int C, bool f32, const float* gamma, const float* beta, float eps,
                  const float* w_head, const float* b_head, const int32_t* labels, float* xhat, float* z, float* logits,
                  float* dlogits, float* dz, float* loss_rows, void* dx, float* dw, float* db, float* dgamma, float* dbeta,
                  float* loss, hipStream_t s);
void extract_cls(const void* x, int B, int T, int D, bool f32, float* out, hipStream_t s);
// rows [n, row_bytes] -> rows 0, every, 2 every, ... of dst (row_bytes: a multiple of 4)
void place_rows(const void* rows, int n, size_t row_bytes, int64_t every, void* dst, hipStream_t s);
void place_cls_grad(const float* dxc, int B, int T, int D, bool f32, void* dx, hipStream_t s);
void cross_entropy(const float* logits, const int32_t* labels, int B, int C, float* loss_rows,
                   float* dlogits, float* loss, hipStream_t s);
void mean_sq_loss(const void* x, int64_t n, bool f32, float* partial, float* loss, void* dx,
                  hipStream_t s);
size_t mean_sq_partial_floats();

// ---- mixture-of-experts FFN (bf16) ----------------------------------------------------------------
constexpr int MOE_MAX_EXPERTS = 32, MOE_MAX_TOPK = 4;
// from the router logits [M,E]: the K largest (ties: lower index) in descending order, or the forced
// choice; gates = softmax over the K selected logits
// (of token t: row t * forced_pitch)
void moe_topk(const float* logits, int64_t M, int E, int K, const int32_t* forced, int64_t forced_pitch, int32_t* experts,
              float* gates, hipStream_t s);
// bf16 copy of w_router [D,E] stored [E,D]
void moe_router_copy(const float* w_router, int D, int E, void* t_router, hipStream_t s);
// stable counting sort of the (token, slot) pairs by expert: off[E+1], pos[t*K+s] = row of the pair
// in expert order, perm_tok[row] = t
void moe_sort(const int32_t* experts, int64_t M, int E, int K, int32_t* off, int32_t* pos, int32_t* perm_tok,
              hipStream_t s);
// y[r,:] = x[src[r],:]   (rows of D bf16, D % 8 == 0)
void moe_gather_rows(const void* x, const int32_t* src, int64_t rows, int D, void* y, hipStream_t s);
// x_out[t,:] = res[t,:] + sum_s gates[t,s] * y[pos[t,s],:]   (y: fp32 expert outputs)
void moe_combine(const void* y, const int32_t* pos, const float* gates, const void* res, int64_t M, int D, int K,
                 void* x_out, hipStream_t s);
// backward of moe_combine w.r.t. y and the gates: dy[pos[t,s],:] = gates[t,s] * dx[t,:];
// dgate_s = <dx[t], y[pos[t,s]]>; dsel[t,s] = gates_s (dgate_s - sum_j gates_j dgate_j) (fp32): the gradient at
// the K selected router logits of token t (the other logits get none)
void moe_combine_bwd(const void* dx, const void* y, const int32_t* pos, const int32_t* experts, const float* gates,
                     int64_t M, int D, int E, int K, void* dy, float* dsel, hipStream_t s);
// dW_r[D,E] (fp32) = h^T dlogits with dlogits[t, experts[t,s]] = dsel[t,s] kept in fp32; partial: scratch of
// moe_router_wgrad_partial_floats(D, E) floats; sums in a fixed order
size_t moe_router_wgrad_partial_floats(int D, int E);
void moe_router_wgrad(const void* h, const int32_t* experts, const float* dsel, int64_t M, int D, int E, int K,
                      float* partial, float* dw, hipStream_t s);
// dh[t,:] = sum_s dxg[pos[t,s],:] + sum_s dsel[t,s] * w_router[:, experts[t,s]]
void moe_unpermute_bwd(const void* dxg, const int32_t* pos, const int32_t* experts, const float* dsel,
                       const float* w_router, int64_t M, int D, int E, int K, void* dh, hipStream_t s);

// Update rule of the optimiser kernels.  SGD: g' = g + wd w; mu > 0: m = mu m + g', w -= lr m; else
// w -= lr g'.  AdamW: m = b1 m + (1-b1) g; v = b2 v + (1-b2) g^2; w -= lr ((m/bc1) / (sqrt(v/bc2) + eps)
// + wd w) with bc = 1 - b^t computed on the host.
enum { OPT_SGD = 0, OPT_ADAMW = 1 };
struct OptArgs { int kind = OPT_SGD; float lr = 0.f, mu = 0.f, wd = 0.f, b1 = 0.f, b2 = 0.f, eps = 0.f, bc1 = 1.f, bc2 = 1.f; };

// A table of weight matrices handled by one launch: bf16 copies (straight and / or transposed) of each, optionally after an optimiser
// update; and of small tensors without copies (biases, LayerNorm parameters, the head), which only get the update.  The table travels as a
// kernel argument (< 4 KB): six dense blocks, or six and the head, fit.
constexpr int OPT_MATS = 24, OPT_VECS = 52;
struct MatEntry { float* w; const float* g; float* m; float* v2; bf16* s; bf16* t; int rows, cols, count; };      // count: matrices behind each other
struct VecEntry { float* w; const float* g; float* m; float* v2; int64_t n; };
struct OptTable {
  MatEntry mat[OPT_MATS];
  VecEntry vec[OPT_VECS];
  int mat_start[OPT_MATS], vec_start[OPT_VECS];      // first workgroup of each (vectors: behind the matrices')
  int mats = 0, vecs = 0, mat_blocks = 0, vec_blocks = 0;
};
// an entry more; a full table is run first
void opt_add_mat(OptTable& t, const MatEntry& e, bool update, const OptArgs& o, hipStream_t s);
void opt_add_vec(OptTable& t, const VecEntry& e, bool update, const OptArgs& o, hipStream_t s);
void opt_run(OptTable& t, bool update, const OptArgs& o, hipStream_t s);      // leaves it empty
// fp32 C[M,N] = A.B (+bias) for tiny problems (the classification head)
void gemm_small_f32(const GemmDesc& g, hipStream_t s);

}  // namespace bsr
