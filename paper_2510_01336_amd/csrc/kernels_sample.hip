// Rejection-sampling acceptance (App. G): exit distributions, the accept test and the draws.
// All random numbers are inputs (uniform in [0, 1)); nothing here generates any.
#include "kernels.h"
#include "draw.h"

#define EE_SAMPLE_THREADS 1024

__device__ inline float block_reduce_max(float v, float* sh) {
  for (int s = 1; s < 64; s <<= 1) v = fmaxf(v, __shfl_xor(v, s, 64));
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  float r = sh[0];
  for (int w = 1; w < EE_SAMPLE_THREADS / 64; ++w) r = fmaxf(r, sh[w]);
  __syncthreads();
  return r;
}
// sum in a fixed order (lanes by butterfly, then the sixteen wave sums one after the other)
__device__ inline float block_reduce_sum(float v, float* sh) {
  for (int s = 1; s < 64; s <<= 1) v += __shfl_xor(v, s, 64);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  float r = 0.f;
  for (int w = 0; w < EE_SAMPLE_THREADS / 64; ++w) r += sh[w];
  __syncthreads();
  return r;
}

// ---- rows of a vocabulary: who reads what ----
// One workgroup of sixteen waves per row; wave w owns the contiguous tokens [w*R, (w+1)*R), R a multiple of 256, and walks them
// 256 at a time, four per lane (one 16-byte load where the rows allow it).  For the inverse CDF a wave keeps the weight of each
// of its (up to 64 groups of) chunks in the lane of that number, so the chunk that holds a draw is found with shuffles and only
// that chunk is read again.  One compute unit takes in about 60 GB/s, which is what bounds these kernels (32000 tokens: 128
// KB, 2 us); the first version let every thread walk a contiguous strip of its own (uncoalesced) and one thread add up
// 1024 strip sums: 67 us a draw at 32000 tokens.
struct RowSpan { int i0, i1, per; };       // this wave's tokens, chunks per group
__device__ inline RowSpan row_span(int vocab) {
  const int w = threadIdx.x >> 6, R = ((vocab + 16 * 256 - 1) / (16 * 256)) * 256;
  RowSpan r;
  r.i0 = min(vocab, w * R); r.i1 = min(vocab, (w + 1) * R);
  r.per = (R / 256 + 63) / 64;
  return r;
}
// four consecutive elements from i (those below n; the others 0); VEC: i and the row are 16-byte aligned
template <bool VEC>
__device__ inline float4 load4(const float* __restrict__ x, int i, int n) {
  if (VEC && i + 3 < n) return *(const float4*)(x + i);
  return make_float4(i < n ? x[i] : 0.f, i + 1 < n ? x[i + 1] : 0.f, i + 2 < n ? x[i + 2] : 0.f, i + 3 < n ? x[i + 3] : 0.f);
}
__device__ inline float wave_sum(float v) {
  for (int s = 1; s < 64; s <<= 1) v += __shfl_xor(v, s, 64);
  return v;
}
// inclusive sum over the lanes below and this one
__device__ inline float wave_scan(float v) {
  const int lane = threadIdx.x & 63;
  for (int s = 1; s < 64; s <<= 1) {
    const float o = __shfl_up(v, s, 64);
    if (lane >= s) v += o;
  }
  return v;
}
// The draw: first token with weight whose cumulative weight exceeds u * (sum of weights).  group: the weight of chunk group `lane` of this
// wave, last: this thread's last token with weight (-1: none); weight(i) gives four consecutive weights.
struct DrawShared { float tot[16]; int last[16]; int tok; };
template <typename W>
__device__ inline int draw_token(const RowSpan& sp, float group, int last, float u, DrawShared& sh, W weight) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const float incl = wave_scan(group);
  for (int s = 1; s < 64; s <<= 1) last = max(last, __shfl_xor(last, s, 64));
  if (lane == 63) { sh.tot[w] = incl; sh.last[w] = last; }
  if (threadIdx.x == 0) sh.tok = -1;
  __syncthreads();
  float total = 0.f;
  int end = -1;
  for (int k = 0; k < 16; ++k) { total += sh.tot[k]; end = max(end, sh.last[k]); }
  const float target = u * total;
  float pre = 0.f;
  int h = -1;
  for (int k = 0; k < 16 && h < 0; ++k) {
    if (pre + sh.tot[k] > target) h = k;
    else pre += sh.tot[k];
  }
  if (h == w) {
    const unsigned long long over = __ballot(draw_admits_group(pre + incl, group, target)), held = __ballot(group > 0.f);
    // (none: the wave's own sum passes the target but no group's prefix does -- its last group with weight)
    const int gl = over ? __ffsll((long long)over) - 1 : 63 - __clzll((long long)held);
    float run = pre + (gl ? __shfl(incl, gl - 1, 64) : 0.f);
    int tok = -1, seen = -1;                            // (seen: the group's last token with weight, should rounding pass the target by)
    for (int c = 0; c < sp.per && tok < 0; ++c) {
      const int i = sp.i0 + (gl * sp.per + c) * 256 + 4 * lane;
      if (i - 4 * lane >= sp.i1) break;
      const float4 x = weight(i);
      const float s3 = ((x.x + x.y) + x.z) + x.w, inc = wave_scan(s3);
      const int k = draw_among_four(run + (inc - s3), x, target);
      const unsigned long long hit = __ballot(k < 4);
      if (hit) {
        const int l = __ffsll((long long)hit) - 1;
        tok = __shfl(i + k, l, 64);
      }
      const int mine = draw_last_of_four(x);
      if (mine >= 0) seen = i + mine;
      run += __shfl(inc, 63, 64);
    }
    for (int s = 1; s < 64; s <<= 1) seen = max(seen, __shfl_xor(seen, s, 64));
    if (lane == 0) sh.tok = tok >= 0 ? tok : seen;
  }
  __syncthreads();
  return sh.tok >= 0 ? sh.tok : end;                     // rounding at the very end of the interval: the last token with weight
}

// p = softmax(logits) per row; row r of `in` (stride vocab floats) -> row out_idx[r] (or r) + out_add of `out`, and of `out2` if
// set.  In place when in == out with the same row mapping.  DRAW: also draws the row's token from p with u[row_seq[r]*u_stride + j].
template <bool VEC, bool DRAW>
__global__ __launch_bounds__(EE_SAMPLE_THREADS) void softmax_rows_kernel(const float* in, float* out, const int* out_idx, int out_add,
                                                                        float* out2, const int* out2_idx, int vocab,
                                                                        const float* __restrict__ u, int u_stride, int j,
                                                                        const int* __restrict__ row_seq, int* tok_next, int* draft_out,
                                                                        int stride) {
  __shared__ float sh[EE_SAMPLE_THREADS / 64];
  __shared__ DrawShared ds;
  const int r = blockIdx.x, lane = threadIdx.x & 63;
  const float* x = in + (size_t)r * vocab;
  float* y = out + (size_t)((out_idx ? out_idx[r] : r) + out_add) * vocab;
  float* y2 = out2 ? out2 + (size_t)out2_idx[r] * vocab : nullptr;
  const RowSpan sp = row_span(vocab);
  float mx = -INFINITY;
#pragma unroll 4
  for (int i = sp.i0 + 4 * lane; i < sp.i1; i += 256) {
    const float4 v = load4<VEC>(x, i, sp.i1);
    mx = fmaxf(mx, fmaxf(fmaxf(v.x, i + 1 < sp.i1 ? v.y : v.x), fmaxf(i + 2 < sp.i1 ? v.z : v.x, i + 3 < sp.i1 ? v.w : v.x)));
  }
  mx = block_reduce_max(mx, sh);
  float sum = 0.f;
#pragma unroll 4
  for (int i = sp.i0 + 4 * lane; i < sp.i1; i += 256) {
    const float4 v = load4<VEC>(x, i, sp.i1);
    sum += (__expf(v.x - mx) + (i + 1 < sp.i1 ? __expf(v.y - mx) : 0.f)) + ((i + 2 < sp.i1 ? __expf(v.z - mx) : 0.f) + (i + 3 < sp.i1 ? __expf(v.w - mx) : 0.f));
  }
  sum = block_reduce_sum(sum, sh);
  const float inv = 1.0f / sum;
  float group = 0.f;
  int last = -1, chunk = 0;
  for (int c0 = sp.i0; c0 < sp.i1; c0 += 1024) {              // four chunks in flight; the whole wave walks every one (the sums use all lanes)
    float4 v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = load4<VEC>(x, c0 + 256 * q + 4 * lane, sp.i1);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int i = c0 + 256 * q + 4 * lane;
      float4 p = make_float4(0.f, 0.f, 0.f, 0.f);
      if (i < sp.i1) p.x = __expf(v[q].x - mx) * inv;
      if (i + 1 < sp.i1) p.y = __expf(v[q].y - mx) * inv;
      if (i + 2 < sp.i1) p.z = __expf(v[q].z - mx) * inv;
      if (i + 3 < sp.i1) p.w = __expf(v[q].w - mx) * inv;
      if (VEC && i + 3 < sp.i1) {
        *(float4*)(y + i) = p;
        if (y2) *(float4*)(y2 + i) = p;
      } else {
        const float e[4] = {p.x, p.y, p.z, p.w};
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if (i + k < sp.i1) { y[i + k] = e[k]; if (y2) y2[i + k] = e[k]; }
      }
      if (DRAW) {
        const float sm = wave_sum((p.x + p.y) + (p.z + p.w));
        if (chunk / sp.per == lane) group += sm;
        last = p.w > 0.f ? i + 3 : (p.z > 0.f ? i + 2 : (p.y > 0.f ? i + 1 : (p.x > 0.f ? i : last)));
        ++chunk;
      }
    }
  }
  if (DRAW) {
    __syncthreads();                                     // (and the row is complete: a chunk of it is read again)
    const int b = row_seq[r];
    const int tok = draw_token(sp, group, last, u[(size_t)b * u_stride + j], ds, [&](int i) { return load4<VEC>(y, i, sp.i1); });
    if (threadIdx.x == 0) { tok_next[r] = tok; draft_out[b * stride + j] = tok; }
  }
}
static bool rows_aligned(int vocab, const float* a, const float* b, const float* c) {
  return vocab % 4 == 0 && (((uintptr_t)a | (uintptr_t)b | (uintptr_t)c) & 15) == 0;
}
void k_softmax_rows(hipStream_t st, const float* in, float* out, const int* out_idx, int out_add, float* out2, const int* out2_idx, int M, int vocab) {
  if (M <= 0) return;
  if (rows_aligned(vocab, in, out, out2))
    hipLaunchKernelGGL((softmax_rows_kernel<true, false>), dim3(M), dim3(EE_SAMPLE_THREADS), 0, st, in, out, out_idx, out_add, out2, out2_idx,
                       vocab, nullptr, 0, 0, nullptr, nullptr, nullptr, 0);
  else
    hipLaunchKernelGGL((softmax_rows_kernel<false, false>), dim3(M), dim3(EE_SAMPLE_THREADS), 0, st, in, out, out_idx, out_add, out2, out2_idx,
                       vocab, nullptr, 0, 0, nullptr, nullptr, nullptr, 0);
}
void k_softmax_draw(hipStream_t st, const float* in, float* out, const int* out_idx, int out_add, int M, int vocab, const float* u, int u_stride,
                    int j, const int* row_seq, int* tok_next, int* draft_out, int stride) {
  if (M <= 0) return;
  if (rows_aligned(vocab, in, out, nullptr))
    hipLaunchKernelGGL((softmax_rows_kernel<true, true>), dim3(M), dim3(EE_SAMPLE_THREADS), 0, st, in, out, out_idx, out_add, nullptr, nullptr,
                       vocab, u, u_stride, j, row_seq, tok_next, draft_out, stride);
  else
    hipLaunchKernelGGL((softmax_rows_kernel<false, true>), dim3(M), dim3(EE_SAMPLE_THREADS), 0, st, in, out, out_idx, out_add, nullptr, nullptr,
                       vocab, u, u_stride, j, row_seq, tok_next, draft_out, stride);
}

// The accept tests of one block per sequence (one wavefront each): candidate j, drawn from row
// draft_row0 + j of the draft distributions, is accepted when u < min(1, p_target / p_draft) at that token;
// n_accept = number of leading accepted candidates.
__global__ void rs_accept_kernel(const float* __restrict__ Pt, const float* __restrict__ Pd, int pd_rows_per_seq, int vocab,
                                 const int* seq_row0, const int* seq_m, const int* cand, const int* n_cand, int cand_stride,
                                 const float* __restrict__ u_acc, int u_stride, int* n_accept) {
  const int b = blockIdx.x, lane = threadIdx.x;
  const int m = seq_m[b];
  if (m == 0) { if (lane == 0) n_accept[b] = -1; return; }
  const int nc = n_cand[b], row0 = seq_row0[b];
  int a = nc;
  for (int j0 = 0; j0 < nc; j0 += 64) {
    const int j = j0 + lane;
    bool rej = false;
    if (j < nc) {
      const int tok = cand[b * cand_stride + j];
      const float pt = Pt[(size_t)(row0 + j) * vocab + tok], pd = Pd[((size_t)b * pd_rows_per_seq + j) * vocab + tok];
      rej = !(u_acc[(size_t)b * u_stride + j] < fminf(1.0f, pt / pd));
    }
    const unsigned long long mask = __ballot(rej);
    if (mask) { a = j0 + __ffsll((long long)mask) - 1; break; }
  }
  if (lane == 0) n_accept[b] = a;
}
void k_rs_accept(hipStream_t st, const float* Pt, const float* Pd, int pd_rows_per_seq, int vocab, const CallMeta& meta,
                 int cand_stride, int B, const float* u_acc, int u_stride, int* n_accept) {
  hipLaunchKernelGGL(rs_accept_kernel, dim3(B), dim3(64), 0, st, Pt, Pd, pd_rows_per_seq, vocab, meta.seq_row0, meta.seq_m,
                     meta.cand, meta.n_cand, cand_stride, u_acc, u_stride, n_accept);
}

// after the accept tests: the replacement from the residual distribution at the first rejected position, or,
// when every candidate was accepted and the block has one more row, the target's own next token
// -- one inverse-CDF draw per sequence; weight(i) = max(0, target - draft) or the target's own probability
template <bool VEC>
__global__ __launch_bounds__(EE_SAMPLE_THREADS) void rs_draw_kernel(const float* __restrict__ Pt, const float* __restrict__ Pd,
                                                                    int pd_rows_per_seq, int vocab, const int* seq_row0,
                                                                    const int* seq_m, const int* n_cand, const int* n_accept,
                                                                    const float* __restrict__ u_res, int* __restrict__ result) {
  __shared__ DrawShared ds;
  const int b = blockIdx.x, lane = threadIdx.x & 63;
  const int m = seq_m[b], a = n_accept[b], nc = n_cand[b];
  int* next_tok = result + gridDim.x;
  if (threadIdx.x == 0) result[b] = a;                   // (-1 for a sequence that takes no part)
  if (m == 0) { if (threadIdx.x == 0) next_tok[b] = -1; return; }
  if (a >= m) { if (threadIdx.x == 0) next_tok[b] = -1; return; }      // all accepted and no further row
  const float* A = Pt + (size_t)(seq_row0[b] + a) * vocab;
  const float* Bd = a < nc ? Pd + ((size_t)b * pd_rows_per_seq + a) * vocab : nullptr;
  const RowSpan sp = row_span(vocab);
  auto weight = [&](int i) {
    float4 x = load4<VEC>(A, i, sp.i1);
    if (Bd) {
      const float4 q = load4<VEC>(Bd, i, sp.i1);
      x = make_float4(fmaxf(0.f, x.x - q.x), fmaxf(0.f, x.y - q.y), fmaxf(0.f, x.z - q.z), fmaxf(0.f, x.w - q.w));
    }
    return x;
  };
  float group = 0.f;
  int last = -1, chunk = 0;
  for (int c0 = sp.i0; c0 < sp.i1; c0 += 1024) {         // four chunks in flight
    float4 x[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) x[q] = weight(c0 + 256 * q + 4 * lane);      // (0 past the end)
#pragma unroll
    for (int q = 0; q < 4; ++q, ++chunk) {
      const int i = c0 + 256 * q + 4 * lane;
      const float sm = wave_sum((x[q].x + x[q].y) + (x[q].z + x[q].w));
      if (chunk / sp.per == lane) group += sm;
      last = x[q].w > 0.f ? i + 3 : (x[q].z > 0.f ? i + 2 : (x[q].y > 0.f ? i + 1 : (x[q].x > 0.f ? i : last)));
    }
  }
  const int tok = draw_token(sp, group, last, u_res[b], ds, weight);
  if (threadIdx.x == 0) next_tok[b] = tok;
}
void k_rs_draw(hipStream_t st, const float* Pt, const float* Pd, int pd_rows_per_seq, int vocab, const CallMeta& meta, int B,
               const int* n_accept, const float* u_res, int* result) {
  if (rows_aligned(vocab, Pt, Pd, nullptr))
    hipLaunchKernelGGL((rs_draw_kernel<true>), dim3(B), dim3(EE_SAMPLE_THREADS), 0, st, Pt, Pd, pd_rows_per_seq, vocab, meta.seq_row0,
                       meta.seq_m, meta.n_cand, n_accept, u_res, result);
  else
    hipLaunchKernelGGL((rs_draw_kernel<false>), dim3(B), dim3(EE_SAMPLE_THREADS), 0, st, Pt, Pd, pd_rows_per_seq, vocab, meta.seq_row0,
                       meta.seq_m, meta.n_cand, n_accept, u_res, result);
}
