// Launchers of the HIP kernels (internal).  All work is enqueued on `st`; nothing synchronises.
#pragma once
#include "common.h"
#include "strips.h"

// ---- dtype-independent ---------------------------------------------------------------------
// per sequence: a = number of leading j < n_cand[b] with cand[b][j] == v[row0[b]+j];
// next = v[row0+a] if a < m[b] else -1.  Sequences with m[b] == 0 report (-1, -1).
void k_accept(hipStream_t st, const int* v, const CallMeta& meta, int cand_stride, int B, int* n_accept, int* next_tok);
// Sequential drafting and decoding, one row per sequence: the arg max kernels hand a row's token on as the next input
// (tok_next[r]) and to the caller (draft_out[row_seq[r]*stride + j]); tok_next == null: nothing to hand on.
struct TakeToken { int* tok_next = nullptr; int* draft_out = nullptr; const int* row_seq = nullptr; int stride = 0, j = 0; };
__device__ inline void take_token(const TakeToken& t, int r, int tok) {
  if (!t.tok_next) return;
  t.tok_next[r] = tok;
  t.draft_out[t.row_seq[r] * t.stride + t.j] = tok;
}
// dst[0..n) <- src (host memory, read before the call returns; n and dst whole int4s); false: too many, nothing done
bool k_store_meta(hipStream_t st, const int* src, int* dst, int n);
void k_fill_nan_dead_kv(hipStream_t st, bool bf16, void* kv, const int* pages, int n_owned_pages, int len,
                        int layer0, int layer1, int n_pages, int n_kv, int D);
void k_read_kv(hipStream_t st, bool bf16, const void* kv, const int* pages, int layer, int pos0, int n,
               int n_pages, int n_kv, int D, float* k_out, float* v_out);
void k_write_kv(hipStream_t st, bool bf16, void* kv, const int* pages, int layer, int pos0, int n, int n_pages, int n_kv, int D,
                const float* k_in, const float* v_in);

// ---- fp32 reference-precision path (EE_F32 models) -----------------------------------------
// rows of a pass into X (embedding of tok, rows[row_idx], or as they stand), cs[r][i] = (cos, sin)(pos_r * inv_freq[i]), rowinfo[r] =
// (first q-tile of the row's sequence, row inside the sequence, KV page, slot in page)
void f32_begin_pass(hipStream_t st, const float* emb, const int* tok, const float* rows, const int* row_idx, float* X, int M, int d,
                    const CallMeta& mt, int pos_add, const double* inv_freq, float2* cs, int half, int pps, int4* rowinfo);
struct F32Out {
  float* Y = nullptr; int ldy = 0;                                    // target rows (F_QKV: Q rows [M][Hq][D])
  float* Y2 = nullptr; const int* y2_idx = nullptr; int y2_add = 0;   // F_ADD: the new rows also go to Y2[y2_idx[row] + y2_add]
  const float2* cs = nullptr; const int4* rowinfo = nullptr;          // F_QKV
  int Hq = 0, Hkv = 0, D = 0, layer = 0, n_pages = 0;
  float* kv = nullptr;
};
// Every projection reads X through an RMSNorm with gain g (null: as it is); W row-major [N][K].
// Y[m][n] (+)= sum_k x[m][k] W[n][k]
void f32_gemm(hipStream_t st, const float* X, int ldx, const float* g, float eps, const float* W, float* Y, int ldy, int M, int N, int K, bool add,
              float* Y2 = nullptr, const int* y2_idx = nullptr, int y2_add = 0);
// H = silu(gate) * up; W: gate and up rows in alternating blocks of 16
void f32_gate_up(hipStream_t st, const float* X, const float* g, float eps, const float* W, float* H, int M, int F, int d);
// fused QKV: rotated Q rows, rotated K and V into their cache pages
void f32_qkv(hipStream_t st, const float* X, const float* g, float eps, const float* W, int M, int d, const F32Out& out);
void f32_attention(hipStream_t st, const float* Q, const float* kv, const CallMeta& meta, int pos_add, int M, int Hq, int Hkv,
                   int D, int layer, int n_pages, int pages_per_seq, int max_ctx, float* out);
void f32_argmax(hipStream_t st, const float* logits, int M, int V, int* v, const TakeToken& take);

// ---- bf16 MFMA path (EE_BF16 models) ---------------------------------------------------------
enum { EPI_ADD = 0, EPI_SWIGLU = 1, EPI_ARGMAX = 2, EPI_ROPE = 3 };
// Deferred RMSNorm of a GEMM's activation operand: the rows hold bf16(x * gain) and the per-row factor
// rsqrt(mean(x^2) + eps) is applied to the fp32 accumulators in the epilogue (it commutes with the
// product).  ssq holds partial sums of squares [n_part][stride] left by the GEMM that produced x;
// null = the operand is already fully normalised.
struct NormIn {
  const float* ssq = nullptr; int n_part = 0, stride = 0; float inv_d = 0.f, eps = 0.f;
  const float* inv_rms = nullptr;   // row-tiled GEMM only: the factors themselves, reduced from ssq beforehand
};
// EPI_ADD extra output: the updated residual rows as the next GEMM's operand, bf16(x * g) in fragment
// layout, plus this tile's partial sums of squares ssq[tile][row].
struct NormOut {
  const float* g = nullptr; bf16_t* xn = nullptr; int ktiles = 0; float* ssq = nullptr; int stride = 0;
};
// EPI_ROPE (fused QKV projection): rotate Q and K, write Q tiles for the attention kernel and K/V into
// their cache pages.
struct RopeOut {
  const float2* cs = nullptr;   // [rows][D/2] (cos, sin) of every row's position
  const int4* rowinfo = nullptr;   // [rows] (first q-tile of the row's sequence, row inside the sequence, KV page, slot in page)
  int Hq = 0, Hkv = 0, D = 0, layer = 0, n_pages = 0, total_qt = 0;
  bf16_t *Q = nullptr, *kv = nullptr;
};
struct GemmOut {
  float* Y = nullptr; int ldy = 0;        // EPI_ADD: residual stream, Y = R + product (row-major fp32; null: only the next operand); EPI_ARGMAX: optional logits
  const float* R = nullptr;               // EPI_ADD: the rows added to (usually Y itself; null: none)
  float* Y2 = nullptr; const int* y2_idx = nullptr; int y2_add = 0;   // EPI_ADD: the new rows also go to Y2[y2_idx[row] + y2_add] (kept hidden rows of an exit)
  bf16_t* H = nullptr; int h_ktiles = 0;  // EPI_SWIGLU target (fragment layout)
  float* pmax = nullptr; int* pidx = nullptr; int pstride = 0;   // EPI_ARGMAX partials [row][pstride >= ntiles]
  NormIn nin;
  NormOut nout;
  RopeOut rope;
};
// Y^T tile = W tile (A operand) x X^T (B operand); W in fragment layout, A in that of the activations.  Up to 32 rows, row0 .. row0+M-1
// of the operand (row0 a multiple of 16), in the launch shape of strip_shape.
void bf16_gemm(hipStream_t st, int epi, const bf16_t* W, int ntiles, int ktiles, const bf16_t* A, int M, int N, const GemmOut& out, int row0 = 0);
// Launch timing: while this points to a pair of events, the next skinny-GEMM launch attaches them to the dispatch
// itself (hipExtLaunchKernelGGL), so that they hold the kernel's own start and end rather than the times at which
// two marker packets around it were processed; the launcher sets `used`.
struct LaunchEvents { hipEvent_t start, stop; bool used; };
extern LaunchEvents* g_launch_events;
extern int g_attn_pages_override;   // <= 0: pages per KV split chosen from the call's shape; else that many (test hook: batch and solo runs then cut their contexts alike)
extern int g_attn_form;              // -1: attention kernel chosen from the call's shape; else that one (ATTN_*) on every call (test hook)
extern int g_rows_wide;              // 1: gate/up and exit head beyond 256 rows run in blocks of 256 rows; 0: in passes of up to 512 rows (test hook)
extern int g_block_tiles;            // > 0: every call that the skinny kernel does not have to serve runs blocked with that many weight tiles per workgroup, plus 100 times the row tiles if not 16 (test hook)
extern int g_rows_blocks_override;   // -1: built-in choice between K shares and row blocks; else 0, or row tiles per block (+100: eight weight tiles per workgroup)
size_t bf16_gemm_rows_scratch_floats(int ntiles, int ktiles);
// Whether bf16_gemm serves a call of M rows, else bf16_gemm_rows.  While a test hook forces a form of the latter, it gets every call of
// more than 16 rows of a matrix of 128 MB and more.
bool bf16_takes_strips(int ntiles, int ktiles, int M);
// Row-tiled variant for more than 16 rows (rows start at row 0 of the operand; the kernels read whole row tiles up to the
// next of 64, 128, 192, 256, 384, 512 rows, beyond 512 up to whole parts of 512, which the operand buffer must hold).
// scratch: bf16_gemm_rows_scratch_floats() floats for this shape (may be null when that is 0); inv_rms: inv_cap (at least
// 512) floats of scratch for the deferred RMSNorm factors; a call of more rows is cut into parts of that size.
// Returns how many partial sums of squares per row an EPI_ADD call with nout left (n_part of the next NormIn).
int bf16_gemm_rows(hipStream_t st, int epi, const bf16_t* W, int ntiles, int ktiles, const bf16_t* A, int M, int N,
                   const GemmOut& out, float* scratch, float* inv_rms, int inv_cap);
// out row r (GEMM operand) <- RMSNorm of row idx[r] of X with gain g
void bf16_rmsnorm(hipStream_t st, const float* X, const int* idx, const float* g, float eps, bf16_t* out, int ktiles, int M, int d);
// Rows row_idx[0..M) of X to `rows`, and q-tiles qt_src[0..n_qt) of Q [kv head][total_qt tiles] to Qt [kv head][n_qt]
void bf16_gather_tail(hipStream_t st, const float* X, const int* row_idx, int M, int d, float* rows, const bf16_t* Q, const int* qt_src, int n_qt,
                      int total_qt, int Hkv, int D, bf16_t* Qt);
// Opens a pass over layers in one launch: row r of X <- embedding of tok[r] (emb set), rows[row_idx[r]] (rows set) or
// itself; out <- its RMSNorm with gain g as a GEMM operand; cs / rowinfo as f32_begin_pass fills them.
void bf16_begin_pass(hipStream_t st, const bf16_t* emb, const int* tok, const float* rows, const int* row_idx, float* X,
                     const float* g, float eps, bf16_t* out, int ktiles, int M, int d, const CallMeta& mt, int pos_add,
                     const double* inv_freq, float2* cs, int half, int pps, int4* rowinfo);
struct AttnScratch { float* part_o; float* part_ml; int max_splits; };
// Attention kernel and KV splits of a call (the same for all its layers), chosen from the sequence ends (kv_end[b] = first
// position past the block, 0 for a sequence not taking part): every split takes `per` pages, the longest sequence has nsplit.
enum { ATTN_RING = 0, ATTN_BLOCK, ATTN_TILE };
struct AttnPlan { int kind, per, nsplit; };
AttnPlan bf16_attention_plan(const int* kv_end, const int* seq_m, int B, int Hq, int Hkv, int max_splits);
void bf16_attention(hipStream_t st, const AttnPlan& plan, const bf16_t* Q, const bf16_t* kv, const CallMeta& meta, int pos_add, int B,
                    int max_m, int total_qt, int Hq, int Hkv, int D, int layer, int n_pages, int pages_per_seq, const AttnScratch& scr,
                    bf16_t* out, int out_ktiles);
void bf16_argmax_reduce(hipStream_t st, const float* pmax, const int* pidx, int ntiles, int pstride, int M, int* v, const TakeToken& take);

// ---- rejection-sampling acceptance (kernels_sample.hip) ----
// out (and out2, if set) <- softmax of the rows of `in`; k_softmax_draw also draws one token per row from it
void k_softmax_rows(hipStream_t st, const float* in, float* out, const int* out_idx, int out_add, float* out2, const int* out2_idx, int M, int vocab);
void k_softmax_draw(hipStream_t st, const float* in, float* out, const int* out_idx, int out_add, int M, int vocab, const float* u, int u_stride,
                    int j, const int* row_seq, int* tok_next, int* draft_out, int stride);
void k_rs_accept(hipStream_t st, const float* Pt, const float* Pd, int pd_rows_per_seq, int vocab, const CallMeta& meta,
                 int cand_stride, int B, const float* u_acc, int u_stride, int* n_accept);
void k_rs_draw(hipStream_t st, const float* Pt, const float* Pd, int pd_rows_per_seq, int vocab, const CallMeta& meta, int B,
               const int* n_accept, const float* u_res, int* result);   // result: n_accept [B], then the drawn tokens [B]
