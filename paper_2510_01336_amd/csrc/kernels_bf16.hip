// bf16 MFMA path for gfx950: weight-streaming skinny GEMM with fused epilogues, k-query
// causal-in-block GQA attention over the paged KV cache (split over the KV axis), RMSNorm and
// RoPE + KV append producing MFMA-ready operand layouts.
//
// Everything is built around v_mfma_f32_16x16x32_bf16 (D = A*B + C, 16x16 output, K = 32):
//   A operand: lane l holds A[l%16][8*(l/16) .. +7]      B operand: lane l holds B[8*(l/16)..+7][l%16]
//   C/D:       lane l holds D[4*(l/16) + v][l%16], v = 0..3
// All operands are stored in HBM already in that per-lane order ("fragment layout", common.h), so a
// wavefront fetches an operand tile as one fully coalesced 1 KiB load straight into registers; no
// LDS staging or transposition is needed anywhere on the streaming path.
#include "kernels.h"
#include "norm_factor.h"
#include <hip/hip_ext.h>
#include <cmath>
#include <type_traits>

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
__device__ inline f32x4 mfma16(u32x4 a, u32x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
__device__ inline f32x4 mfma16(uint4 a, uint4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
// two fp32 -> packed bf16 pair (lo in bits 0..15), round to nearest even: one v_cvt_pk_bf16_f32
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
__device__ inline uint32_t pack2(float lo, float hi) {
  const f32x2 v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

// ---------------------------------------------------------------------------------------------
// RMSNorm of listed rows: fp32 row idx[r] in, bf16 fragment-layout row r out (the operand of an exit head that serves only
// the rows that decide a token)
// ---------------------------------------------------------------------------------------------
// One workgroup per row; the row is read once as float4 into registers (all loads issued before the
// first use), reduced, scaled, and written as 8-byte bf16 quads (4 consecutive k share a fragment lane).
template <int CH>   // float4 chunks per thread: d <= 4 * 256 * CH
__global__ __launch_bounds__(256) void bf16_rmsnorm_kernel(const float* __restrict__ X, const int* __restrict__ idx,
                                                           const float* __restrict__ g, float eps, bf16_t* __restrict__ out, int ktiles, int d) {
  __shared__ float part[4];
  const int r = blockIdx.x, nch = d >> 2;
  const float4* x4 = (const float4*)(X + (size_t)idx[r] * d);
  const float4* g4 = (const float4*)g;
  float4 xv[CH], gv[CH];
#pragma unroll
  for (int i = 0; i < CH; ++i) {
    const int c = threadIdx.x + i * 256;
    xv[i] = c < nch ? x4[c] : make_float4(0.f, 0.f, 0.f, 0.f);
    gv[i] = c < nch ? g4[c] : make_float4(0.f, 0.f, 0.f, 0.f);
  }
  float ss = 0.f;
#pragma unroll
  for (int i = 0; i < CH; ++i) ss += xv[i].x * xv[i].x + xv[i].y * xv[i].y + xv[i].z * xv[i].z + xv[i].w * xv[i].w;
  for (int o = 32; o > 0; o >>= 1) ss += __shfl_down(ss, o, 64);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = ss;
  __syncthreads();
  const float inv = 1.0f / sqrtf((part[0] + part[1] + part[2] + part[3]) / (float)d + eps);
#pragma unroll
  for (int i = 0; i < CH; ++i) {
    const int c = threadIdx.x + i * 256;
    if (c < nch) {
      uint2 pk = make_uint2(pack2(xv[i].x * inv * gv[i].x, xv[i].y * inv * gv[i].y),
                            pack2(xv[i].z * inv * gv[i].z, xv[i].w * inv * gv[i].w));
      *(uint2*)(out + act_offset(r, c * 4, ktiles)) = pk;
    }
  }
}
void bf16_rmsnorm(hipStream_t st, const float* X, const int* idx, const float* g, float eps, bf16_t* out, int ktiles, int M, int d) {
  // d is a multiple of 16 for bf16 models (checked at model load), so float4 access is aligned
  if (d <= 1024) hipLaunchKernelGGL((bf16_rmsnorm_kernel<1>), dim3(M), dim3(256), 0, st, X, idx, g, eps, out, ktiles, d);
  else if (d <= 4096) hipLaunchKernelGGL((bf16_rmsnorm_kernel<4>), dim3(M), dim3(256), 0, st, X, idx, g, eps, out, ktiles, d);
  else hipLaunchKernelGGL((bf16_rmsnorm_kernel<16>), dim3(M), dim3(256), 0, st, X, idx, g, eps, out, ktiles, d);
}

// The first kernel of a pass over layers, one workgroup per row: brings the row into the residual stream X -- from the
// embedding table by token, from a buffer of kept hidden rows by index, or leaves it where it is --, writes its
// RMSNorm as the first projection's operand, and fills the row's rotary table and epilogue lookups on the side: first q-tile
// of its sequence, row inside the sequence, KV page and slot of its position, so that the QKV epilogue of every layer finds
// them with one row-indexed load instead of a chain of dependent ones.  One launch where the pass used to open with three.
template <int CH>
__global__ __launch_bounds__(256) void bf16_begin_pass_kernel(const bf16_t* __restrict__ emb, const int* __restrict__ tok,
                                                              const float* __restrict__ rows, const int* __restrict__ row_idx,
                                                              float* __restrict__ X, const float* __restrict__ g, float eps,
                                                              bf16_t* __restrict__ out, int ktiles, int d, const int* row_pos,
                                                              int pos_add, const double* inv_freq, float2* cs, int half,
                                                              const int* row_seq, const int* seq_row0, const int* seq_qt0,
                                                              const int* block_table, int pps, int4* rowinfo) {
  __shared__ float part[4];
  const int r = blockIdx.x, nch = d >> 2;
  const float4* g4 = (const float4*)g;
  float4 xv[CH], gv[CH];
  if (emb) {
    const uint2* e2 = (const uint2*)(emb + (size_t)tok[r] * d);          // four bf16 per chunk
#pragma unroll
    for (int i = 0; i < CH; ++i) {
      const int c = threadIdx.x + i * 256;
      const uint2 e = c < nch ? e2[c] : make_uint2(0u, 0u);
      xv[i] = make_float4(__uint_as_float(e.x << 16), __uint_as_float(e.x & 0xffff0000u), __uint_as_float(e.y << 16),
                          __uint_as_float(e.y & 0xffff0000u));
    }
  } else {
    const float4* x4 = (const float4*)((rows ? rows : X) + (size_t)(row_idx ? row_idx[r] : r) * d);
#pragma unroll
    for (int i = 0; i < CH; ++i) {
      const int c = threadIdx.x + i * 256;
      xv[i] = c < nch ? x4[c] : make_float4(0.f, 0.f, 0.f, 0.f);
    }
  }
#pragma unroll
  for (int i = 0; i < CH; ++i) {
    const int c = threadIdx.x + i * 256;
    gv[i] = c < nch ? g4[c] : make_float4(0.f, 0.f, 0.f, 0.f);
  }
  const int pos = row_pos[r] + pos_add;
  for (int f = threadIdx.x; f < half; f += 256) {     // rotary angles in double: at position 32768 an fp32 product pos*freq is off by ~2e-3 rad
    double sn, cn;
    sincos((double)pos * inv_freq[f], &sn, &cn);
    cs[(size_t)r * half + f] = make_float2((float)cn, (float)sn);
  }
  if (threadIdx.x == 0) {
    const int sq = row_seq[r];
    rowinfo[r] = make_int4(seq_qt0[sq], r - seq_row0[sq], block_table[sq * pps + pos / EE_PAGE], pos % EE_PAGE);
  }
  if (emb || rows) {
    float4* xo = (float4*)(X + (size_t)r * d);
#pragma unroll
    for (int i = 0; i < CH; ++i) {
      const int c = threadIdx.x + i * 256;
      if (c < nch) xo[c] = xv[i];
    }
  }
  float ss = 0.f;
#pragma unroll
  for (int i = 0; i < CH; ++i) ss += xv[i].x * xv[i].x + xv[i].y * xv[i].y + xv[i].z * xv[i].z + xv[i].w * xv[i].w;
  for (int o = 32; o > 0; o >>= 1) ss += __shfl_down(ss, o, 64);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = ss;
  __syncthreads();
  const float inv = 1.0f / sqrtf((part[0] + part[1] + part[2] + part[3]) / (float)d + eps);
#pragma unroll
  for (int i = 0; i < CH; ++i) {
    const int c = threadIdx.x + i * 256;
    if (c < nch) {
      uint2 pk = make_uint2(pack2(xv[i].x * inv * gv[i].x, xv[i].y * inv * gv[i].y),
                            pack2(xv[i].z * inv * gv[i].z, xv[i].w * inv * gv[i].w));
      *(uint2*)(out + act_offset(r, c * 4, ktiles)) = pk;
    }
  }
}
void bf16_begin_pass(hipStream_t st, const bf16_t* emb, const int* tok, const float* rows, const int* row_idx, float* X,
                     const float* g, float eps, bf16_t* out, int ktiles, int M, int d, const CallMeta& mt, int pos_add,
                     const double* inv_freq, float2* cs, int half, int pps, int4* rowinfo) {
#define BEGIN_PASS(CH_)                                                                                                       \
  hipLaunchKernelGGL((bf16_begin_pass_kernel<CH_>), dim3(M), dim3(256), 0, st, emb, tok, rows, row_idx, X, g, eps, out, ktiles, d,  \
                     mt.row_pos, pos_add, inv_freq, cs, half, mt.row_seq, mt.seq_row0, mt.seq_qt0, mt.block_table, pps, rowinfo)
  if (d <= 1024) BEGIN_PASS(1);
  else if (d <= 4096) BEGIN_PASS(4);
  else BEGIN_PASS(16);
#undef BEGIN_PASS
}

// Moves the rows of a context build's last layer that have a reader to the front (a workgroup per row or q-tile): plain copies, bound by
// the launch (512 rows and 128 q-tiles of the 8B width, 12.6 MB read and written, 6.8 us).
__global__ __launch_bounds__(256) void gather_tail_kernel(const float4* __restrict__ X, const int* __restrict__ row_idx, int M, int d4, float4* __restrict__ rows,
                                                          const uint4* __restrict__ Q, const int* __restrict__ qt_src, int n_qt, int total_qt, int Hkv,
                                                          int tile, uint4* __restrict__ Qt) {
  const int r = blockIdx.x;
  if (r < M) {
    const float4* src = X + (size_t)row_idx[r] * d4;
    for (int c = threadIdx.x; c < d4; c += 256) rows[(size_t)r * d4 + c] = src[c];
  } else {
    const int t = r - M, from = qt_src[t];
    for (int i = threadIdx.x; i < Hkv * tile; i += 256)
      Qt[((size_t)(i / tile) * n_qt + t) * tile + i % tile] = Q[((size_t)(i / tile) * total_qt + from) * tile + i % tile];
  }
}
void bf16_gather_tail(hipStream_t st, const float* X, const int* row_idx, int M, int d, float* rows, const bf16_t* Q, const int* qt_src, int n_qt,
                      int total_qt, int Hkv, int D, bf16_t* Qt) {
  hipLaunchKernelGGL(gather_tail_kernel, dim3(M + n_qt), dim3(256), 0, st, (const float4*)X, row_idx, M, d / 4, (float4*)rows, (const uint4*)Q, qt_src, n_qt,
                     total_qt, Hkv, D * 2, (uint4*)Qt);
}

// ---------------------------------------------------------------------------------------------
// Skinny GEMM  Y[m][n] = sum_k X[m][k] W[n][k],  M <= 16*MT rows per launch, weights streamed once.
// A strip is one 16-row weight tile over the whole K.  A wave takes NS strips and a share of K (ksplit waves of the workgroup share
// it out in contiguous chunks) and streams them (1 KiB per MFMA step) through two register sets of U k-tiles that take turns (one in
// flight while the other is multiplied); the partial 16x16 tiles are then summed through LDS in a fixed order (deterministic), the
// strips dealt round the waves for that and for the epilogue.  Every strip is complete in itself (see phys_row), so strips can be
// dealt to any number of waves and workgroups: strip_shape gives every compute unit the same number of them.
// The MFMA computes Y^T = W X^T so that a lane ends up with 4 consecutive n of one row m.
//
// Epilogues (everything between two projections is fused here, so a layer is five launches, six when the attention is split over the KV axis and merged):
//   EPI_ADD     residual add into the fp32 stream; optionally emits the next projection's operand
//               bf16(x_new * gain) and this tile's partial sum of squares per row (deferred RMSNorm)
//   EPI_SWIGLU  silu(gate) * up  -> bf16 operand of the down projection
//   EPI_ROPE    rotary embedding of Q and K; Q tiles for the attention kernel; K, V into cache pages
//   EPI_ARGMAX  per-row (max, arg max) of the tile (+ optional fp32 logits)
// Every epilogue first applies the operand's deferred RMSNorm factor (NormIn).
// ---------------------------------------------------------------------------------------------
// ---- epilogue of one 16 x 16 output tile (or tile pair), shared by the skinny and the row-tiled GEMM ----
// A lane of the epilogue wave holds, for row m = mt*16 + lane%16, the four consecutive outputs
// n = 16*tile + 4*(lane/16) .. +3.  Tiles of the paired epilogues hold eight features and their partners (up for gate, the other
// rotary half for Q/K/V; see phys_row): the upper half of the wave holds the partners of the lower half's outputs.
struct EpiPre {            // operands of the epilogue that do not depend on the product
  float4 res, gnext;       // EPI_ADD: residual row slice, gains of the next operand
  float4 rc[2];            // EPI_ROPE: (cos, sin) of the lane's two or four rotary pairs
  int r_a, r_b;            // EPI_ROPE: Q heads: (global q-tile, row in tile); K/V heads: (page, position in page)
                           // EPI_ADD: r_a = row of the second destination
};

// Deals the pairs of one tile (NF = 2), or of two neighbouring ones (NF = 4: wider stores), to all lanes: lo[i], hi[i] = output
// pair_feature<NF> + i behind the first tile's first feature and its partner.
template <int NF>
__device__ inline void pair_up(const f32x4& a, const f32x4& b, float sc, float (&lo)[NF], float (&hi)[NF]) {
  typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));
#pragma unroll
  for (int i = 0; i < NF; ++i) {
    const u32x2_t r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a[i] * sc), __float_as_uint((NF == 2 ? a[2 + i] : b[i]) * sc), false, false);
    lo[i] = __uint_as_float(r[0]); hi[i] = __uint_as_float(r[1]);
  }
}
// Kernels that stage weight tiles in LDS can do without: of a pair of tiles t and t + 1 they fetch the sixteen features into
// one slot and their partners into the next, so that a lane finds both in its two accumulators (QKV of 96 x 16 tiles at 512
// rows 30.6 -> 28.4 us, 8B gate/up at 2048 with the stores below 374.8 -> 368.6).  Lane `lane` of slot `slot` fetches unit paired_unit of tile
// (slot & ~1) + paired_tile:
__device__ inline int paired_tile(int lane) { return (lane >> 3) & 1; }
__device__ inline int paired_unit(int lane, int slot) { return (lane >> 4) * 16 + (lane & 7) + 8 * (slot & 1); }
template <int NF>
__device__ inline int pair_feature(int lane) { return NF == 2 ? ((lane >> 4) & 1) * 4 + (lane >> 5) * 2 : (lane >> 4) * 4; }
template <int NF>
__device__ inline void store_bf16(bf16_t* p, const float (&x)[NF]) {
  if constexpr (NF == 2) *(uint32_t*)p = pack2(x[0], x[1]);
  else *(uint2*)p = make_uint2(pack2(x[0], x[1]), pack2(x[2], x[3]));
}

template <int EPI, int NF = 2>
__device__ inline void epi_prefetch(EpiPre& p, const GemmOut& out, int task, int row, bool ok, int lane) {
  const int g = lane >> 4;
  p.res = p.gnext = make_float4(0.f, 0.f, 0.f, 0.f);
  p.rc[0] = p.rc[1] = make_float4(1.f, 0.f, 1.f, 0.f);
  p.r_a = p.r_b = 0;
  if (EPI == EPI_ADD) {
    const int n = task * 16 + 4 * g;
    if (ok && out.R) p.res = *(const float4*)(out.R + (size_t)row * out.ldy + n);
    if (out.nout.xn) p.gnext = *(const float4*)(out.nout.g + n);
    if (out.Y2 && ok) p.r_a = out.y2_idx[row] + out.y2_add;
  }
  if (EPI == EPI_ROPE && ok) {
    const RopeOut& R = out.rope;
    const int half = R.D >> 1, tph = R.D >> 4;
    const int h = task / tph, f = (task % tph) * 8 + pair_feature<NF>(lane);
    const int4 ri = R.rowinfo[row];              // (every operand here is indexed by the row alone: no dependent loads)
    if (h < R.Hq + R.Hkv) {
      const float4* c4 = (const float4*)(R.cs + (size_t)row * half + f);
      p.rc[0] = c4[0];
      if constexpr (NF == 4) p.rc[1] = c4[1];
    }
    if (h < R.Hq) {
      const int q = ri.y * (R.Hq / R.Hkv) + h % (R.Hq / R.Hkv);
      p.r_a = ri.x + (q >> 4); p.r_b = q & 15;
    } else {
      p.r_a = ri.z; p.r_b = ri.w;
    }
  }
}

// Deferred RMSNorm: row factors from the producer's partial sums of squares [partial][row], in a fixed order.  A lane loads four
// rows (lane % 4) of every 16th partial (lane / 4); the sixteen lanes of a row quad then add up theirs.
// sum over the lanes of equal lane % 4, delivered to all of them, neighbours first
__device__ inline float quad_lane_sum(float x) {
  typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));
  x += __shfl_xor(x, 4, 64);
  x += __shfl_xor(x, 8, 64);
  u32x2_t r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
template <int NT>
struct NormPartials { float4 t[NT][4]; };      // 64 partials of NT row tiles (row0 + 16 * step * i, i < n), requested ahead of their use
template <int NT>
__device__ inline void norm_request(NormPartials<NT>& q, const NormIn& nin, int row0, int step, int n, int c0, int lane) {
  const float* p = nin.ssq + row0 + 4 * (lane & 3);
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int i = 0; i < NT; ++i)
      q.t[i][j] = *(const float4*)(p + (size_t)min(c0 + (lane >> 2) + 16 * j, nin.n_part - 1) * nin.stride + 16 * step * min(i, n - 1));
}
// Factors sc[i] of rows row0 + 16 * step * i + lane % 16 (row0 a multiple of 16; i < n of NT); q: partials 0..63.  The row tiles
// go side by side, so the chain is one tile's.
template <int NT>
__device__ inline void norm_factors(float (&sc)[NT], NormPartials<NT>& q, const NormIn& nin, int row0, int step, int n, int lane) {
  float4 sv[NT];
#pragma unroll
  for (int i = 0; i < NT; ++i) sv[i] = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int c0 = 0;;) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (c0 + (lane >> 2) + 16 * j < nin.n_part) {
#pragma unroll
        for (int i = 0; i < NT; ++i) { sv[i].x += q.t[i][j].x; sv[i].y += q.t[i][j].y; sv[i].z += q.t[i][j].z; sv[i].w += q.t[i][j].w; }
      }
    c0 += 64;
    if (c0 >= nin.n_part) break;
    norm_request<NT>(q, nin, row0, step, n, c0, lane);
  }
  const int mc = lane & 15;
#pragma unroll
  for (int i = 0; i < NT; ++i) {
    sv[i].x = quad_lane_sum(sv[i].x); sv[i].y = quad_lane_sum(sv[i].y); sv[i].z = quad_lane_sum(sv[i].z); sv[i].w = quad_lane_sum(sv[i].w);
    // lanes with lane % 4 == q now hold rows 4q .. 4q+3
    const float a = __shfl(sv[i].x, mc >> 2, 64), b = __shfl(sv[i].y, mc >> 2, 64), c = __shfl(sv[i].z, mc >> 2, 64), e = __shfl(sv[i].w, mc >> 2, 64);
    const float ss = (mc & 2) ? ((mc & 1) ? e : c) : ((mc & 1) ? b : a);
    sc[i] = 1.0f / sqrtf(ss * nin.inv_d + nin.eps);
  }
}

// The paired epilogues on a lane's features lo and their partners hi.  NF = 2: of one tile; 4: of tiles `tile` and `tile` + 1
template <int EPI, int NF>
__device__ inline void epi_store_pairs(float (&lo)[NF], float (&hi)[NF], const EpiPre& p, const GemmOut& out, int tile, int row, int lane) {
  if (EPI == EPI_SWIGLU) {
    const int f = tile * 8 + pair_feature<NF>(lane);     // h[m][f ..] = silu(gate) * up
    float h[NF];
#pragma unroll
    for (int v = 0; v < NF; ++v) h[v] = lo[v] / (1.0f + __expf(-lo[v])) * hi[v];
    store_bf16<NF>(out.H + act_offset(row, f, out.h_ktiles), h);
  } else {
    // head h, features f .. and their partners f + D/2 ..
    const RopeOut& R = out.rope;
    const int D = R.D, half = D >> 1, tph = D >> 4;
    const int h = tile / tph, f = (tile % tph) * 8 + pair_feature<NF>(lane);
    if (h < R.Hq + R.Hkv) {
#pragma unroll
      for (int v = 0; v < NF; ++v) {
        const float4 t = p.rc[v >> 1];
        const float c = v & 1 ? t.z : t.x, s = v & 1 ? t.w : t.y, a = lo[v], b = hi[v];
        lo[v] = fmaf(a, c, -(b * s));      // (spelled out: the same rounding in every kernel)
        hi[v] = fmaf(b, c, a * s);
      }
    }
    if (h < R.Hq) {
      const int kvh = h / (R.Hq / R.Hkv), q15 = p.r_b;
      const size_t qtile = ((size_t)kvh * R.total_qt + p.r_a) * (D >> 5);
      const int d1 = f + half;
      store_bf16<NF>(R.Q + ((qtile + (f >> 5)) * 64 + ((f & 31) >> 3) * 16 + q15) * 8 + (f & 7), lo);
      store_bf16<NF>(R.Q + ((qtile + (d1 >> 5)) * 64 + ((d1 & 31) >> 3) * 16 + q15) * 8 + (d1 & 7), hi);
    } else {
      const int page = p.r_a, pp = p.r_b;
      if (h < R.Hq + R.Hkv) {
        bf16_t* slab = R.kv + kv_slab(R.layer, page, h - R.Hq, R.n_pages, R.Hkv, D);
        store_bf16<NF>(slab + k_page_off(pp, f, D), lo);
        store_bf16<NF>(slab + k_page_off(pp, f + half, D), hi);
      } else {
        bf16_t* slab = R.kv + kv_slab(R.layer, page, h - R.Hq - R.Hkv, R.n_pages, R.Hkv, D) + EE_PAGE * D;
#pragma unroll
        for (int v = 0; v < NF; v += 2) {
          const uint32_t wl = pack2(lo[v], lo[v + 1]), wh = pack2(hi[v], hi[v + 1]);
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            slab[v_page_off(pp, f + v + j)] = (bf16_t)(wl >> (16 * j));
            slab[v_page_off(pp, f + half + v + j)] = (bf16_t)(wh >> (16 * j));
          }
        }
      }
    }
  }
}

// tiles as they lie in memory (eight features and their partners), NF as above (NF = 4: the next one's accumulators in acc1)
template <int EPI, int NF>
__device__ inline void epi_apply_tiles(const f32x4& acc0, const f32x4& acc1, float sc, const EpiPre& p, const GemmOut& out, int tile, int row, bool ok, int lane) {
  float lo[NF], hi[NF];
  pair_up<NF>(acc0, acc1, sc, lo, hi);
  if (ok) epi_store_pairs<EPI, NF>(lo, hi, p, out, tile, row, lane);
}
// tiles `tile` and `tile` + 1, fetched as paired_unit says
template <int EPI>
__device__ inline void epi_apply_pair(const f32x4& acc0, const f32x4& acc1, float sc, const EpiPre& p, const GemmOut& out, int tile, int row, bool ok, int lane) {
  float lo[4], hi[4];
#pragma unroll
  for (int v = 0; v < 4; ++v) { lo[v] = acc0[v] * sc; hi[v] = acc1[v] * sc; }
  if (ok) epi_store_pairs<EPI, 4>(lo, hi, p, out, tile, row, lane);
}

// SwiGLU of the pair for two row tiles at once: lanes 16..31 and 48..63 give their features to the lanes below them and take over the
// second row tile, so that every lane stores a whole 16-byte unit.  Halves of units, in runs of 64 bytes, made gate/up launches with
// little K slower than with an operand in fragment order: 86 x 8 tiles at 512 / 2048 rows 17.9 / 69.9 us, 17.4 / 67.4 in fragment order, 16.2 /
// 62.6 as it is now.
__device__ inline void epi_swiglu_two_rows(const f32x4& gate0, const f32x4& up0, float sc0, const f32x4& gate1, const f32x4& up1, float sc1, const GemmOut& out,
                                           int tile, int row0, bool ok0, int row1, bool ok1, int lane) {
  typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));
  float h0[4], h1[4];
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const float a = gate0[v] * sc0, b = gate1[v] * sc1;
    h0[v] = a / (1.0f + __expf(-a)) * (up0[v] * sc0);
    h1[v] = b / (1.0f + __expf(-b)) * (up1[v] * sc1);
  }
  const u32x2_t x = __builtin_amdgcn_permlane16_swap(pack2(h0[0], h0[1]), pack2(h1[0], h1[1]), false, false);
  const u32x2_t y = __builtin_amdgcn_permlane16_swap(pack2(h0[2], h0[3]), pack2(h1[2], h1[3]), false, false);
  const bool second = lane & 16;
  if (second ? ok1 : ok0) *(uint4*)(out.H + act_offset(second ? row1 : row0, tile * 8 + (lane >> 5) * 8, out.h_ktiles)) = make_uint4(x[0], y[0], x[1], y[1]);
}

// sc: the row's deferred RMSNorm factor (1 when the operand was already normalised)
template <int EPI>
__device__ inline void epi_apply(const f32x4& acc0, float sc, const EpiPre& p, const GemmOut& out, int task,
                                 int row, bool ok, int N, int lane, float* ss_out = nullptr) {
  const int g = lane >> 4;
  if (EPI == EPI_ADD) {
    const int n = task * 16 + 4 * g;
    float4 r = make_float4(acc0[0] * sc, acc0[1] * sc, acc0[2] * sc, acc0[3] * sc);
    r.x += p.res.x; r.y += p.res.y; r.z += p.res.z; r.w += p.res.w;
    if (out.Y && ok) *(float4*)(out.Y + (size_t)row * out.ldy + n) = r;
    if (out.Y2 && ok) *(float4*)(out.Y2 + (size_t)p.r_a * out.ldy + n) = r;
    if (out.nout.xn) {
      const float4 gn = p.gnext;
      if (ok) *(uint2*)(out.nout.xn + act_offset(row, n, out.nout.ktiles)) = make_uint2(pack2(r.x * gn.x, r.y * gn.y), pack2(r.z * gn.z, r.w * gn.w));
      float ss = ok ? (r.x * r.x + r.y * r.y) + (r.z * r.z + r.w * r.w) : 0.f;
      ss += __shfl_xor(ss, 16, 64);
      ss += __shfl_xor(ss, 32, 64);
      if (ss_out) *ss_out = ss;                // (the caller adds up several tiles)
      else if (g == 0 && ok) out.nout.ssq[(size_t)task * out.nout.stride + row] = ss;      // (a full block may visit tiles without rows, see block_full)
    }
  } else if (EPI == EPI_SWIGLU || EPI == EPI_ROPE) {
    epi_apply_tiles<EPI, 2>(acc0, acc0, sc, p, out, task, row, ok, lane);
  } else {   // EPI_ARGMAX: per-row (max, arg max) over this tile's 16 outputs; lowest index wins ties
    float best = -INFINITY; int bi = 0x7fffffff;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int n = task * 16 + 4 * g + v;
      const float t = acc0[v] * sc;
      if (n < N) {
        if (out.Y && ok) out.Y[(size_t)row * out.ldy + n] = t;
        if (t > best) { best = t; bi = n; }
      }
    }
#pragma unroll
    for (int sh = 16; sh <= 32; sh <<= 1) {
      const float ob = __shfl_xor(best, sh, 64); const int oi = __shfl_xor(bi, sh, 64);
      if (ob > best || (ob == best && oi < bi)) { best = ob; bi = oi; }
    }
    if (g == 0 && ok) {
      out.pmax[(size_t)row * out.pstride + task] = best;
      out.pidx[(size_t)row * out.pstride + task] = bi;
    }
  }
}

template <int MT, int NS, int U>
struct Frags {
  u32x4 w[NS][U];
  u32x4 x[MT][U];
};

// Requests the fragments of k-tiles kt .. kt+U-1 (indices past `last` repeat the last k-tile: valid memory; the
// caller leaves those out of the product).  Nothing here touches a loaded value, so the wave does not wait.
template <int MT, int NS, int U>
__device__ inline void load_frags(Frags<MT, NS, U>& f, const u32x4* const (&wp)[NS], const u32x4* const (&ap)[MT], int kt, int last) {
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int k = min(kt + u, last);
#pragma unroll
    for (int s = 0; s < NS; ++s) f.w[s][u] = __builtin_nontemporal_load(&wp[s][(size_t)k * 64]);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) f.x[mt][u] = ap[mt][(size_t)k * 64];
  }
}
// acc += the product over the k-tiles kt .. kt+U-1 held in f; GUARD: only those below kt1 (kt and kt1 must be
// uniform in a way the compiler can see, see the kernel)
template <int MT, int NS, int U, bool GUARD>
__device__ inline void mma_frags(f32x4 (&acc)[NS][MT], const Frags<MT, NS, U>& f, int kt, int kt1) {
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (!GUARD || kt + u < kt1) {         // (uniform)
#pragma unroll
      for (int s = 0; s < NS; ++s)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[s][mt] = mfma16(f.w[s][u], f.x[mt][u], acc[s][mt]);
    }
}

template <int MT, int EPI, int NS, int U, bool HALF = false>
__global__ __launch_bounds__(64 * EE_MAX_WAVES) void gemm_skinny_kernel(const uint4* __restrict__ W, int ktiles, int ntiles,
                                                                        const uint4* __restrict__ A, int row0, int M, int N,
                                                                        GemmOut out, int ksplit) {
  __shared__ f32x4 red[EE_MAX_WAVES][NS * MT][64];
  __shared__ __align__(16) float ssq_red[EE_MAX_WAVES][MT * 16];
  // The wave's number is taken through a scalar register: the compiler then knows that everything derived from it (the
  // task, the K share and above all the conditions around the MFMAs of a short last group) is uniform and branches
  // on it.  A condition it takes for divergent it may turn into an EXEC mask without a branch -- and the matrix
  // instructions ignore EXEC, so a masked-off MFMA would still add its product.
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = blockDim.x >> 6;
  const int tasks = nw / ksplit, task0 = blockIdx.x * tasks * NS, strip0 = task0 + wave / ksplit * NS, kpart = wave % ksplit;
  // HALF: two workgroups of one XCD share 2 * NS - 1 strips, NS - 1 whole ones each and half of the last: four features and their partners,
  // whose rows the lanes of the other four repeat.
  static_assert(!HALF || (NS > 1 && EPI == EPI_ROPE), "whole strips and a half");
  const int half = HALF ? half_of(blockIdx.x) : 0;
  auto strip_at = [&](int i) { return HALF ? half_strip_at(blockIdx.x, i, NS) : task0 + i; };      // i-th strip of the workgroup
  const int per = (ktiles + ksplit - 1) / ksplit;
  const int kt0 = kpart * per, kt1 = min(ktiles, kt0 + per);

  f32x4 acc[NS][MT];
#pragma unroll
  for (int s = 0; s < NS; ++s)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[s][mt] = f32x4{0.f, 0.f, 0.f, 0.f};

  const bool stream = (HALF ? strip_at(0) : strip0) < ntiles && kt0 < kt1;
  const int mc = lane & 15;
  const u32x4 *wp[NS], *ap[MT];
#pragma unroll
  for (int s = 0; s < NS; ++s)
    wp[s] = (const u32x4*)W + (size_t)min(HALF ? strip_at(s) : strip0 + s, ntiles - 1) * ktiles * 64 + (HALF && s == NS - 1 ? (lane & 0x3b) + 4 * half : lane);
  // (rows past the last repeat it: the quads behind the last row's are not fetched)
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) ap[mt] = (const u32x4*)A + (size_t)((row0 >> 4) + mt) * ktiles * 64 + act_unit(max(0, min(mc, M - 1 - 16 * mt)), lane >> 4);
  Frags<MT, NS, U> cur;

  // Order of the requests: the partial sums of squares of the deferred RMSNorm (contiguous shares of the workgroup's waves, looked
  // at behind the K loop), the first weight fragments, the epilogue's operands.
  const bool normed = out.nin.ssq != nullptr;
  const int np = normed ? out.nin.n_part : 0, cp = (np + nw - 1) / nw, cw = wave * cp, ce = min(np, cw + cp);
  // strip whose epilogue this wave runs first
  const int own = ksplit == 1 ? strip0 : strip_at(wave);
  const bool owner = own < ntiles && (ksplit == 1 || wave < tasks * NS);
  // lane of the tile whose outputs this one holds (every second row of lanes of the half strip repeats the one before it: no results)
  const int elane = HALF && wave == NS - 1 ? (lane & 0x2f) + 16 * half : lane;
  const bool eok = !(HALF && wave == NS - 1 && (lane & 16));
  EpiPre pre[MT];
  NormPartials<MT> part;
  if (normed) norm_request<MT>(part, out.nin, row0, 1, MT, cw, lane);
  if (stream) load_frags<MT, NS, U>(cur, wp, ap, kt0, kt1 - 1);
  if (owner) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) epi_prefetch<EPI>(pre[mt], out, own, row0 + mt * 16 + mc, eok && mt * 16 + mc < M, elane);
  }

  // Two register sets of fragments take turns: while one is multiplied the other is in flight, and the next request
  // for a set goes out as soon as its MFMAs are issued.
  if (stream) {
    // Groups of U k-tiles; only the last one can be short.  In the loop every fragment requested is multiplied, with
    // no condition in between -- a request whose data might go unused would make the compiler drain the load counter
    // before the registers are requested again, and with it the set in flight.
    Frags<MT, NS, U> oth;
    const int last = kt1 - 1;
    int kt = kt0;
    for (; kt + 2 * U < kt1; kt += 2 * U) {
      load_frags<MT, NS, U>(oth, wp, ap, kt + U, last);
      mma_frags<MT, NS, U, false>(acc, cur, kt, kt1);
      load_frags<MT, NS, U>(cur, wp, ap, kt + 2 * U, last);
      mma_frags<MT, NS, U, false>(acc, oth, kt + U, kt1);
    }
    if (kt + U < kt1) {                  // two groups left
      load_frags<MT, NS, U>(oth, wp, ap, kt + U, last);
      mma_frags<MT, NS, U, false>(acc, cur, kt, kt1);
      mma_frags<MT, NS, U, true>(acc, oth, kt + U, kt1);
    } else {
      mma_frags<MT, NS, U, true>(acc, cur, kt, kt1);
    }
  }

  if (normed) {
    float4 sv[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) sv[mt] = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int c0 = cw;;) {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (c0 + (lane >> 2) + 16 * j < ce) {
#pragma unroll
          for (int mt = 0; mt < MT; ++mt) { sv[mt].x += part.t[mt][j].x; sv[mt].y += part.t[mt][j].y; sv[mt].z += part.t[mt][j].z; sv[mt].w += part.t[mt][j].w; }
        }
      c0 += 64;
      if (c0 >= ce) break;
      norm_request<MT>(part, out.nin, row0, 1, MT, c0, lane);      // (more than 64 partials a wave: wide models)
    }
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      const float4 t = make_float4(quad_lane_sum(sv[mt].x), quad_lane_sum(sv[mt].y), quad_lane_sum(sv[mt].z), quad_lane_sum(sv[mt].w));
      if (lane < 4) *(float4*)&ssq_red[wave][mt * 16 + 4 * lane] = t;
    }
  }
  if (ksplit > 1) {
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) red[wave][s * MT + mt][lane] = acc[s][mt];
  }
  if (ksplit > 1 || normed) __syncthreads();   // (uniform; every wave reaches it)
  float sc[MT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    sc[mt] = 1.0f;
    if (normed) {
      float ss = ssq_red[0][mt * 16 + mc];
      for (int w = 1; w < nw; ++w) ss += ssq_red[w][mt * 16 + mc];
      sc[mt] = 1.0f / sqrtf(ss * out.nin.inv_d + out.nin.eps);
    }
  }
  if (ksplit == 1) {
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      if (strip0 + s >= ntiles) continue;
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        const int m = mt * 16 + mc;
        if (s > 0) epi_prefetch<EPI>(pre[mt], out, strip0 + s, row0 + m, m < M, lane);
        epi_apply<EPI>(acc[s][mt], sc[mt], pre[mt], out, strip0 + s, row0 + m, m < M, N, lane);
      }
    }
    return;
  }
  // the strips of the workgroup are dealt round its waves; the K parts of one are added in a fixed order
  for (int i = wave; i < tasks * NS && strip_at(i) < ntiles; i += nw) {      // (HALF: at most one strip a wave)
    const int w0 = i / NS * ksplit, s = i % NS;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      const int m = mt * 16 + mc;
      if (i != wave) epi_prefetch<EPI>(pre[mt], out, strip_at(i), row0 + m, m < M, lane);
      f32x4 sum = red[w0][s * MT + mt][lane];
      for (int w = 1; w < ksplit; ++w) sum += red[w0 + w][s * MT + mt][lane];
      epi_apply<EPI>(sum, sc[mt], pre[mt], out, strip_at(i), row0 + m, eok && m < M, N, elane);
    }
  }
}

// ---------------------------------------------------------------------------------------------
// Row-tiled GEMM for a block of 16 < M <= 512 rows (up to 32 only where that is quicker than the skinny kernel, see
// strips_serve): weights cross HBM once per block, but every weight fragment now
// meets up to 32 row tiles, so the kernel sits near the machine's ridge (M flop per weight byte).
// Workgroup = 8 waves (two per SIMD: one wave alone does not keep a matrix pipe busy) on a group of
// WT = 8 weight tiles (128 output features; 7 where that deals a wide matrix more evenly, see the launcher) and a share of K (grid.y); wave (rq, nh) owns 4 of the tiles and a
// quarter of the TMT row tiles (every fourth one): TMT accumulators.  Row tiles past the last row are neither
// requested nor multiplied.
// Both operands reach LDS by direct global->LDS loads (no staging registers, no LDS store
// instructions): a ring of S stages, one k-tile each (8 KiB of weights + TMT KiB of activations), as many
// as LDS holds, of which up to S-2 are in flight: that is what covers the HBM latency with one workgroup
// per compute unit.  Each wave requests one weight tile and one or two row tiles of every stage; per
// k-tile it waits until its own share of the next stage has landed (the load counter is in order), meets
// the other waves at a barrier -- which also says that everyone is past the MFMAs of the previous stage,
// whose slot the next request then overwrites -- reads the next stage's fragments (1 KiB, lane-linear,
// conflict-free) into the second register set and runs the TMT MFMAs of the current one under them.  The
// loop is unrolled over the ring so that every LDS address is a constant, and indices past the end are
// clamped (only the MFMAs are guarded).
// With grid.y == 1 the epilogue is fused; otherwise fp32 partial tiles go to scratch and
// gemm_rows_reduce_kernel sums the K shares in a fixed order and runs the same epilogue.
// ---------------------------------------------------------------------------------------------
// Whether the partial tiles of K shares stay in the L2 for the reduce kernel, else they stream to memory.  Kernel and reduction inside
// decoding steps of so many rows (kernel trace), us, streamed / kept: 8B QKV at 36 / 64 / 144 / 192 rows 19.6 / 19.0, 20.7 / 20.3, 30.7 / 28.2,
// 34.0 / 33.6; 70B QKV at 144 / 192 / 256 / 512 rows 56.0 / 53.6, 63.2 / 63.4, 71.9 / 73.6, 111.6 / 112.7; 8B O at 36 / 144 15.6 / 14.8, 21.9 / 20.8; 8B
// down at 36 / 96 / 144 / 256 / 512 29.5 / 29.2, 34.6 / 34.9, 38.8 / 37.3, 52.1 / 50.8, 74.8 / 73.5; 70B down at 144 / 256 97.5 / 96.2, 133 / 131.
// So only the widest partial sums, those of QKV beyond 192 rows, are better out of the way.
__device__ inline bool keep_partials(int epi, int M) { return epi != EPI_ROPE || M <= 192; }
// s_waitcnt immediate: at most n vector-memory loads outstanding, all LDS reads done, export counter untouched
__host__ __device__ constexpr int waitcnt_vm_lgkm0(int n) { return (n & 15) | ((n >> 4) << 14) | (7 << 4); }

template <int TMT, int EPI, bool FULL, int TN, int WT = 2 * TN>
__global__ __launch_bounds__(512) void gemm_rows_kernel(const uint4* __restrict__ W, int ktiles, int ntiles,
                                                        const uint4* __restrict__ A, int row0, int M_all, int N, GemmOut out,
                                                        int per, float* __restrict__ partial) {
  // rows row0 .. row0+M_all-1 of the operand (row0 a multiple of 16), of which this workgroup takes the block of
  // TMT*16 rows that blockIdx.z names; the deferred-norm factors and the K-share partials are indexed from row0,
  // everything the epilogue touches by the row itself
  static_assert((TN == 2 || TN == 4) && (WT == 2 * TN || WT == 2 * TN - 1), "weight tiles per wave");
  const int bx = blockIdx.x, rbase = blockIdx.z * (TMT * 16), M = min(M_all - rbase, TMT * 16);
  constexpr int TMW = TMT / 4;                      // row tiles per wave
  static_assert(TMT % 4 == 0 && TMT >= 4 && TMT <= 32, "row tiles split four ways");
  constexpr int STAGE = (WT + TMT) * 64;        // 16-byte units: weight tiles first, then row tiles
  constexpr int S = (160 / (WT + TMT)) & ~1;    // stages in the ring: what 160 KiB of LDS holds (even: fragments alternate between two register sets)
  constexpr int XHI = (TMT + 7) / 8;                // row tiles a wave requests per stage at most: wave, wave+8, ...
  constexpr int LHI = 1 + XHI;                      // requests per stage at most (one weight tile, XHI row tiles)
  static_assert((S - 1) * LHI < 64, "the load counter has six bits");
  __shared__ u32x4 ring[S][STAGE];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wave_s = __builtin_amdgcn_readfirstlane(wave);      // the same number, known to be uniform
  const int rq = wave_s >> 1, nh = wave_s & 1;
  const int rqv = wave >> 1, nhv = wave & 1;                    // the same again from the vector register: one address register
                                                                // serves all LDS reads, the slots being constant offsets from it
  const int nt0 = bx * WT + nh * TN;                      // first weight tile of this wave
  // Row tiles of this wave: TMW in a row when all of them hold rows (FULL: the guards below fold away), else
  // rq, rq+4, ..., so that the tiles past the last row, which are neither requested nor multiplied, are spread
  // over the four wave pairs.  The launcher picks the smallest TMT that holds the rows, so the unused tiles are
  // among the last eight.
  constexpr int MT_STEP = FULL ? 1 : 4;                         // tile of accumulator mt: mt_first + mt * MT_STEP
  const int mt_first = FULL ? rq * TMW : rq;
  const int mt_used = FULL ? TMT : (M + 15) >> 4;
  const int kt0 = blockIdx.y * per, kt1 = min(ktiles, kt0 + per);
  if (kt0 >= kt1) return;                                       // whole workgroup (never with the launcher's shapes)
  const int last = kt1 - 1;

  f32x4 acc[TN][TMW];
#pragma unroll
  for (int tn = 0; tn < TN; ++tn)
#pragma unroll
    for (int mt = 0; mt < TMW; ++mt) acc[tn][mt] = f32x4{0.f, 0.f, 0.f, 0.f};

  // this wave's share of a stage: weight tile `wave` of the group and row tiles wave, wave+8, ... (every
  // wave requests both kinds with the same lead: a wave's load counter is in order, so it could not wait
  // for a recent request without draining all its older ones)
  typedef const __attribute__((address_space(1))) void* gptr_t;
  typedef __attribute__((address_space(3))) void* lptr_t;
  // this wave's last row tile holds rows: XHI requests per stage, else one less; with four weight tiles per
  // workgroup (TN = 2) only the first four waves request one
  const bool hi = (FULL && TMT % 8 == 0) || wave_s + 8 * (XHI - 1) < mt_used;
  const bool wreq = WT >= 8 || wave_s < WT;
  // LDS byte address of this wave's weight tile in stage 0 as a scalar: every request's LDS address is this plus a
  // constant, so none of them occupies a vector register (measured: 3-4 % at 24 and 32 row tiles)
  const unsigned lds0 = __builtin_amdgcn_readfirstlane((unsigned)(size_t)(lptr_t)&ring[0][0]) + 1024u * wave_s;
#define ROWS_LDS(slot_, tile_) ((lptr_t)(size_t)(lds0 + 16u * ((slot_) * STAGE + (tile_) * 64)))
  constexpr int PT = EPI == EPI_SWIGLU || EPI == EPI_ROPE ? 2 : 1;      // tiles the epilogue takes at once
  // (K shares leave their partial tiles as they lie in memory; so does the last of seven tiles, which has no partner here)
  const bool paired = PT == 2 && gridDim.y == 1 && wave_s < (WT & ~1);
  const u32x4* wsrc = (const u32x4*)W + (size_t)min(bx * WT + (paired ? (wave & ~1) + paired_tile(lane) : wave), ntiles - 1) * ktiles * 64 +
                      (paired ? paired_unit(lane, wave) : lane);
  const u32x4* xsrc = (const u32x4*)A + (size_t)(((row0 + rbase) >> 4) + wave) * ktiles * 64 + act_unit(lane & 15, lane >> 4);
  // (weights: streaming hint)
#define ROWS_REQUEST(slot_, kt_)                                                                              \
  do {                                                                                                        \
    const size_t k_ = (size_t)min(kt_, last) * 64;                                                            \
    if (wreq) __builtin_amdgcn_global_load_lds((gptr_t)(wsrc + k_), ROWS_LDS(slot_, 0), 16, 0, 2);                \
    _Pragma("unroll") for (int j = 0; j < XHI - 1; ++j)                                                       \
      __builtin_amdgcn_global_load_lds((gptr_t)(xsrc + (size_t)(8 * j) * ktiles * 64 + k_),                   \
                                       ROWS_LDS(slot_, WT + 8 * j), 16, 0, 0);                            \
    if (hi)                                                                                                   \
      __builtin_amdgcn_global_load_lds((gptr_t)(xsrc + (size_t)(8 * (XHI - 1)) * ktiles * 64 + k_),           \
                                       ROWS_LDS(slot_, WT + 8 * (XHI - 1)), 16, 0, 0);                    \
  } while (0)
#define ROWS_WAIT(stages_)                                                                                    \
  do {                                                                                                        \
    if (wreq && hi) __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0((stages_) * LHI));                            \
    else if (wreq) __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0((stages_) * (LHI - 1)));                       \
    else if (hi) __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0((stages_) * XHI));                               \
    else __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0((stages_) * (XHI - 1)));                                 \
  } while (0)
#define ROWS_READ(buf_, slot_)                                                                               \
  do {                                                                                                        \
    const u32x4* wl_ = &ring[slot_][(nhv * TN) * 64 + lane];                                                  \
    const u32x4* xl_ = &ring[slot_][(WT + (FULL ? rqv * TMW : rqv)) * 64 + lane];                         \
    _Pragma("unroll") for (int tn = 0; tn < TN; ++tn) wf[buf_][tn] = wl_[tn * 64];                            \
    _Pragma("unroll") for (int mt = 0; mt < TMW; ++mt) xf[buf_][mt] = xl_[mt * MT_STEP * 64];                 \
  } while (0)
  u32x4 wf[2][TN], xf[2][TMW];      // fragments of the k-tile being multiplied and of the next one
#pragma unroll
  for (int s = 0; s < S - 1; ++s) ROWS_REQUEST(s, kt0 + s);
  ROWS_WAIT(S - 2);
  __builtin_amdgcn_s_barrier();
  ROWS_READ(0, 0);
  // One k-tile: own share of stage u+1 landed and own fragment reads done; then everybody's, and everybody
  // is past the MFMAs of stage u-1, whose slot the next request overwrites.  The requests and the reads of
  // the next fragments do not depend on this k-tile's MFMAs and ride along with them, one row tile's four
  // MFMAs at a time (the scheduling barriers pin that order): issued in one burst after the barrier, the
  // eight waves' LDS reads would queue up while the matrix pipes sit idle.
#define ROWS_STEP(u_, guard_)                                                                                 \
  do {                                                                                                        \
    ROWS_WAIT(S - 3);                                                                                         \
    __builtin_amdgcn_s_barrier();                                                                             \
    const int cb_ = (u_) & 1, nb_ = cb_ ^ 1, ns_ = ((u_) + 1) % S;                                            \
    ROWS_REQUEST(((u_) + S - 1) % S, kt + (u_) + S - 1);                                                      \
    const u32x4* wl_ = &ring[ns_][(nhv * TN) * 64 + lane];                                                    \
    const u32x4* xl_ = &ring[ns_][(WT + (FULL ? rqv * TMW : rqv)) * 64 + lane];                           \
    const bool on_ = !(guard_) || kt + (u_) < kt1;                                                            \
    __builtin_amdgcn_sched_barrier(0);                                                                        \
    _Pragma("unroll") for (int mt = 0; mt < TMW; ++mt) {                                                      \
      _Pragma("unroll") for (int tn = mt * TN / TMW; tn < (mt + 1) * TN / TMW; ++tn) wf[nb_][tn] = wl_[tn * 64]; \
      xf[nb_][mt] = xl_[mt * MT_STEP * 64];                                                                   \
      if (on_ && (FULL || 4 * mt + 11 < TMT || rq + 4 * mt < mt_used)) {                                      \
        _Pragma("unroll") for (int tn = 0; tn < TN; ++tn) acc[tn][mt] = mfma16(wf[cb_][tn], xf[cb_][mt], acc[tn][mt]); \
      }                                                                                                       \
      __builtin_amdgcn_sched_barrier(0);                                                                      \
    }                                                                                                         \
  } while (0)
  // of the two waves that share a SIMD the hardware favours the older one; the younger four get the higher
  // priority so that both reach the barrier closer together (measured: 1-3 % at 144 rows)
  if (wave_s >= 4) __builtin_amdgcn_s_setprio(2);
  int kt = kt0;
  for (; kt + S <= kt1; kt += S) {
#pragma unroll
    for (int u = 0; u < S; ++u) ROWS_STEP(u, false);
  }
  if (kt < kt1) {                                  // fewer than S k-tiles left: same steps, MFMAs guarded
#pragma unroll
    for (int u = 0; u < S; ++u) ROWS_STEP(u, true);
  }
#undef ROWS_STEP
#undef ROWS_READ
#undef ROWS_WAIT
#undef ROWS_REQUEST
#undef ROWS_LDS
  __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(0));              // requests past the end have landed before the wave moves on

  const int mc = lane & 15;
  if (gridDim.y > 1) {
    // K share: raw accumulator tiles [k share][weight tile][row tile][lane] for the reduce kernel
    f32x4* pp = (f32x4*)partial + (size_t)blockIdx.y * ntiles * TMT * 64 + lane;
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) {
      if (nt0 + tn >= ntiles) continue;
#pragma unroll
      for (int mt = 0; mt < TMW; ++mt)
        if (mt_first + mt * MT_STEP < mt_used) {
          if (keep_partials(EPI, M_all)) pp[((size_t)(nt0 + tn) * TMT + mt_first + mt * MT_STEP) * 64] = acc[tn][mt];
          else __builtin_nontemporal_store(acc[tn][mt], pp + ((size_t)(nt0 + tn) * TMT + mt_first + mt * MT_STEP) * 64);
        }
    }
    return;
  }
  float sc[TMW];        // the rows' deferred RMSNorm factors: reduced beforehand, or here from the producer's partial sums
#pragma unroll
  for (int mt = 0; mt < TMW; ++mt) {
    sc[mt] = 1.0f;
    if (out.nin.inv_rms && mt_first + mt * MT_STEP < mt_used) sc[mt] = out.nin.inv_rms[rbase + min((mt_first + mt * MT_STEP) * 16 + mc, M - 1)];
  }
  const int mt_own = (mt_used - mt_first + MT_STEP - 1) / MT_STEP;      // row tiles of this wave that hold rows
  if (!out.nin.inv_rms && out.nin.ssq && mt_own > 0) {
    NormPartials<TMW> part;
    norm_request<TMW>(part, out.nin, row0 + rbase + mt_first * 16, MT_STEP, min(mt_own, TMW), 0, lane);
    norm_factors<TMW>(sc, part, out.nin, row0 + rbase + mt_first * 16, MT_STEP, min(mt_own, TMW), lane);
  }
#pragma unroll
  for (int t = 0; t < TN; t += PT) {
    const int task = nt0 + t;
    if (task >= ntiles || (WT < 2 * TN && nh && t == TN - 1)) continue;
    const bool lone = PT == 2 && WT < 2 * TN && nh && t == TN - 2;      // (the next tile is another workgroup's)
    constexpr int RT = EPI == EPI_SWIGLU && TMW > 1 ? 2 : 1;            // row tiles it takes at once
    const bool mine = PT == 1 || WT == 2 * TN || task + 1 < ntiles || lane < 32;      // (no next tile: only the lanes of the first one)
#pragma unroll
    for (int mt = 0; mt < TMW; mt += RT) {
      const int m = (mt_first + mt * MT_STEP) * 16 + mc;
      if (mt_first + mt * MT_STEP >= mt_used) continue;
      if constexpr (RT == 2) {
        if (!lone && mt + 1 < TMW) {
          const int m1 = m + 16 * MT_STEP;
          epi_swiglu_two_rows(acc[t][mt], acc[t + 1][mt], sc[mt], acc[t][mt + 1], acc[t + 1][mt + 1], sc[mt + 1], out, task, row0 + rbase + m, m < M && mine,
                              row0 + rbase + m1, m1 < M && mine, lane);
          continue;
        }
      }
#pragma unroll
      for (int r = 0; r < RT; ++r) {
        if (mt + r >= TMW || mt_first + (mt + r) * MT_STEP >= mt_used) continue;
        const int mr = m + 16 * MT_STEP * r;
        EpiPre pre;
        epi_prefetch<EPI, 2 * PT>(pre, out, task, row0 + rbase + mr, mr < M, lane);
        if (lone) epi_apply_tiles<EPI, 2>(acc[t][mt + r], acc[t][mt + r], sc[mt + r], pre, out, task, row0 + rbase + mr, mr < M, lane);
        else if constexpr (PT == 2) epi_apply_pair<EPI>(acc[t][mt + r], acc[t + 1][mt + r], sc[mt + r], pre, out, task, row0 + rbase + mr, mr < M && mine, lane);
        else epi_apply<EPI>(acc[t][mt + r], sc[mt + r], pre, out, task, row0 + rbase + mr, mr < M, N, lane);
      }
    }
  }
}

// ---------------------------------------------------------------------------------------------
// Blocked GEMM for calls of more than 256 rows (context build, large batches): the ring of direct global->LDS stages of
// the kernel above, but the rows are cut into blocks of 16*TMT and the weights into groups of 2*TN tiles, and one launch covers
// all blocks, each XCD on blocks that share weights and rows in its L2 (block_order).  Gate/up and the exit head take blocks of 256 rows; narrow
// matrices those of 256, 192 or 128 rows and 16, 12 or 8 weight tiles that fill the chip without K shares (kNarrowForms).
// What bounds it: with sixteen weight tiles a k-tile is 1024 clocks of MFMAs per SIMD, 128 KiB of LDS traffic (1000 clocks)
// and 32 KiB of requests, and the clock gives way under that load: 8B gate/up at 4096 rows 672 us (1431 TFLOP/s), at 2048 rows 370 (1300), at
// 512 rows in the row-tiled kernel 96 (1253).  (Layers without sampling or profiler on one card; under the profiler, and on other cards, up to 6 % longer.)
// K is never shared out: among calls that run blocked a row's sums run over K in one order, whatever the form and the row
// count.  (Between kernels they do not: skinny, row-tiled and K-share sums differ in order, and the row count decides which
// kernel a call gets.  Within the skinny kernel the order is the matrix's own below 128 MB, see strip_parts.)  K shares of the down projection, tried at
// 1096 rows, were a sixth quicker there and no quicker from 2048; shares
// whose number follows the row count moved the full-depth comparison of a batch with its sequences alone past its bound.
// ---------------------------------------------------------------------------------------------
template <int EPI, int TN, int TMT, bool FULL>
__device__ __forceinline__ void gemm_block_body(u32x4* ring, const uint4* __restrict__ W, int ktiles, int ntiles, const uint4* __restrict__ A,
                                                int row0, int rbase, int M, int N, const GemmOut& out, int bx) {
  constexpr int WT = 2 * TN, TMW = TMT / 4, TILES = WT + TMT, STAGE = TILES * 64;
  static_assert(TMT % 4 == 0 && (EPI != EPI_SWIGLU || TMW % 2 == 0), "row tiles split four ways, and SwiGLU takes two at once");
  constexpr int S = (160 / TILES) & ~1;             // stages in the ring (even: fragments alternate between two register sets)
  constexpr int NJ = block_requests(0, WT, TMT);    // requests per wave and stage at most
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wave_s = __builtin_amdgcn_readfirstlane(wave);
  const int rq = wave_s >> 1, nh = wave_s & 1;
  const int rqv = wave >> 1, nhv = wave & 1;      // (the same from the vector register: one address serves all LDS reads)
  const int nt0 = bx * WT + nh * TN;
  constexpr int MT_STEP = FULL ? 1 : 4;             // a partly filled block deals its row tiles round, a full one in runs
  const int mt_first = FULL ? rq * TMW : rq;
  const int mt_used = FULL ? TMT : (M + 15) >> 4;
  const int last = ktiles - 1;
  f32x4 acc[TN][TMW];
#pragma unroll
  for (int tn = 0; tn < TN; ++tn)
#pragma unroll
    for (int mt = 0; mt < TMW; ++mt) acc[tn][mt] = f32x4{0.f, 0.f, 0.f, 0.f};

  typedef const __attribute__((address_space(1))) void* gptr_t;
  typedef __attribute__((address_space(3))) void* lptr_t;
  const unsigned lds0 = __builtin_amdgcn_readfirstlane((unsigned)(size_t)(lptr_t)ring) + 1024u * wave_s;
  constexpr int PT = EPI == EPI_SWIGLU || EPI == EPI_ROPE ? 2 : 1;      // tiles the epilogue takes at once
  const u32x4* src[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int t = wave_s + 8 * j;
    // (QKV as it lies in memory: paired, 4096 rows took 202 us against 198 at the 8B width)
    const bool paired = EPI == EPI_SWIGLU;
    const int wt = paired ? (t & ~1) + paired_tile(lane) : t;
    const size_t tile = t < WT ? (size_t)min(bx * WT + wt, ntiles - 1) : (size_t)(((row0 + rbase) >> 4) + min(t - WT, (M - 1) >> 4));
    src[j] = (t < WT ? (const u32x4*)W + (paired ? paired_unit(lane, t) : lane) : (const u32x4*)A + act_unit(lane & 15, lane >> 4)) + tile * ktiles * 64;
  }
  // requests of this wave per stage: its tiles that exist and, among the row tiles, hold rows (a prefix of its list)
  const int nreq = block_requests(wave_s, WT, mt_used);
  // The wait chooses among the counts there are, no more: one branch more in every step of a light block (see block_full) costs 4-6 % of
  // calls that end with one (8B gate/up in 12 x 16 tiles at 700 / 960 rows 161 / 238 us with it, 153 / 228 without, down in 16 x 16 at 900 rows 268 / 255).
  constexpr int kLeast = block_requests(7, WT, FULL ? TMT : 1);
  static_assert(kLeast >= 1 && NJ - kLeast <= 3, "waits for NJ, NJ - 1, NJ - 2 and kLeast requests a stage");
#define BLK_REQUEST(slot_, kt_)                                                                               \
  do {                                                                                                        \
    const size_t k_ = (size_t)min(kt_, last) * 64;                                                            \
    _Pragma("unroll") for (int j = 0; j < NJ; ++j)                                                            \
      if (8 * j + 7 < (FULL ? TILES : WT) || j < nreq)                                                        \
        __builtin_amdgcn_global_load_lds((gptr_t)(src[j] + k_), (lptr_t)(size_t)(lds0 + 16u * ((slot_) * STAGE + 8 * j * 64)), 16, 0, 0); \
  } while (0)
#define BLK_WAIT(stages_)                                                                                     \
  do {                                                                                                        \
    if (NJ == kLeast || nreq == NJ) __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0((stages_) * NJ));             \
    else if (NJ - 1 == kLeast || nreq == NJ - 1) __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0((stages_) * (NJ - 1))); \
    else if (NJ - 2 == kLeast || nreq == NJ - 2) __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0((stages_) * (NJ - 2))); \
    else __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0((stages_) * kLeast));                                    \
  } while (0)
  static_assert((S - 1) * NJ < 64, "the load counter has six bits");
  const u32x4* wl0 = ring + (nhv * TN) * 64 + lane;
  const u32x4* xl0 = ring + (WT + (FULL ? rqv * TMW : rqv)) * 64 + lane;
  u32x4 wf[2][TN], xf[2][TMW];
#pragma unroll
  for (int s = 0; s < S - 1; ++s) BLK_REQUEST(s, s);
  BLK_WAIT(S - 2);
  __builtin_amdgcn_s_barrier();
#pragma unroll
  for (int tn = 0; tn < TN; ++tn) wf[0][tn] = wl0[tn * 64];
#pragma unroll
  for (int mt = 0; mt < TMW; ++mt) xf[0][mt] = xl0[mt * MT_STEP * 64];
#define BLK_STEP(u_, guard_)                                                                                  \
  do {                                                                                                        \
    BLK_WAIT(S - 3);                                                                                          \
    __builtin_amdgcn_s_barrier();                                                                             \
    const int cb_ = (u_) & 1, nb_ = cb_ ^ 1, ns_ = ((u_) + 1) % S;                                            \
    BLK_REQUEST(((u_) + S - 1) % S, kt + (u_) + S - 1);                                                       \
    const u32x4* wl_ = wl0 + ns_ * STAGE;                                                                     \
    const u32x4* xl_ = xl0 + ns_ * STAGE;                                                                     \
    const bool on_ = !(guard_) || kt + (u_) < ktiles;                                                            \
    __builtin_amdgcn_sched_barrier(0);                                                                        \
    _Pragma("unroll") for (int mt = 0; mt < TMW; ++mt) {                                                      \
      _Pragma("unroll") for (int tn = mt * TN / TMW; tn < (mt + 1) * TN / TMW; ++tn) wf[nb_][tn] = wl_[tn * 64]; \
      xf[nb_][mt] = xl_[mt * MT_STEP * 64];                                                                   \
      if (on_ && (FULL || rq + 4 * mt < mt_used)) {                                                           \
        _Pragma("unroll") for (int tn = 0; tn < TN; ++tn) acc[tn][mt] = mfma16(wf[cb_][tn], xf[cb_][mt], acc[tn][mt]); \
      }                                                                                                       \
      __builtin_amdgcn_sched_barrier(0);                                                                      \
    }                                                                                                         \
  } while (0)
  if (wave_s >= 4) __builtin_amdgcn_s_setprio(2);
  int kt = 0;
  for (; kt + S <= ktiles; kt += S) {
#pragma unroll
    for (int u = 0; u < S; ++u) BLK_STEP(u, false);
  }
  if (kt < ktiles) {
#pragma unroll
    for (int u = 0; u < S; ++u) BLK_STEP(u, true);
  }
#undef BLK_STEP
#undef BLK_WAIT
#undef BLK_REQUEST
  __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(0));
  const int mc = lane & 15;
#pragma unroll
  for (int t = 0; t < TN; t += PT) {
    const int task = nt0 + t;
    if (task >= ntiles) continue;
#pragma unroll
    for (int mt = 0; mt < TMW; mt += EPI == EPI_SWIGLU ? 2 : 1) {
      const int m = (mt_first + mt * MT_STEP) * 16 + mc;
      if (mt_first + mt * MT_STEP >= mt_used) continue;
      const float sc = out.nin.inv_rms ? out.nin.inv_rms[rbase + min(m, M - 1)] : 1.0f;
      if constexpr (EPI == EPI_SWIGLU) {
        const int m1 = m + 16 * MT_STEP;
        const float sc1 = out.nin.inv_rms ? out.nin.inv_rms[rbase + min(m1, M - 1)] : 1.0f;
        epi_swiglu_two_rows(acc[t][mt], acc[t + 1][mt], sc, acc[t][mt + 1], acc[t + 1][mt + 1], sc1, out, task, row0 + rbase + m, m < M, row0 + rbase + m1, m1 < M, lane);
        continue;
      }
      EpiPre pre;
      epi_prefetch<EPI, 2 * PT>(pre, out, task, row0 + rbase + m, m < M, lane);
      if constexpr (PT == 2) epi_apply_tiles<EPI, 4>(acc[t][mt], acc[t + 1][mt], sc, pre, out, task, row0 + rbase + m, m < M, lane);
      else epi_apply<EPI>(acc[t][mt], sc, pre, out, task, row0 + rbase + m, m < M, N, lane);
    }
  }
}

template <int EPI, int TN, int TMT>
__global__ __launch_bounds__(512) void gemm_block_kernel(const uint4* __restrict__ W, int ktiles, int ntiles, const uint4* __restrict__ A,
                                                         int row0, int M_all, int N, GemmOut out, BlockOrder order) {
  constexpr int TILES = 2 * TN + TMT;
  __shared__ u32x4 ring[((160 / TILES) & ~1) * TILES * 64];
  const BlockPlace at = block_place(order, blockIdx.x);
  if (at.col < 0) return;                           // whole workgroup
  const int bx = at.col, rbase = at.row * (TMT * 16), M = min(M_all - rbase, TMT * 16);
  if (block_full((M + 15) >> 4, TMT)) gemm_block_body<EPI, TN, TMT, true>(ring, W, ktiles, ntiles, A, row0, rbase, M, N, out, bx);
  else gemm_block_body<EPI, TN, TMT, false>(ring, W, ktiles, ntiles, A, row0, rbase, M, N, out, bx);
}

// Sums the K shares of a row tile and runs the epilogue, one wave per task.  Where the partial tiles are kept in the L2
// (keep_partials) the workgroups of a column group (eight weight tiles) run on the XCD that its K shares ran on: workgroup id mod 8,
// where the number of columns is a multiple of 8.  The four waves of a workgroup take four tasks of
// the same row tile and leave one partial sum of squares per row for the four of them, so that the next projection finds a
// quarter of the partials and reads its factors itself (a launch of its own for that took 4.5 us).
#define EE_REDUCE_TASKS 4
template <int EPI>
__global__ __launch_bounds__(64 * EE_REDUCE_TASKS) void gemm_rows_reduce_kernel(const float* __restrict__ partial, int ksplit, int ntiles,
                                                                                int TMT, int row0, int M, int N, GemmOut out) {
  __shared__ float ssq[EE_REDUCE_TASKS][16];
  const int lane = threadIdx.x & 63, mc = lane & 15, wave = threadIdx.x >> 6;
  const int mtiles = (M + 15) >> 4;
  constexpr int QUADS = 2 * EE_ROWS_TN / EE_REDUCE_TASKS;
  int mt, group;
  if (keep_partials(EPI, M)) {
    const int i = blockIdx.x >> 3, column = i / (mtiles * QUADS) * 8 + (blockIdx.x & 7);
    mt = i % mtiles; group = column * QUADS + i / mtiles % QUADS;
  } else {
    mt = blockIdx.x % mtiles; group = blockIdx.x / mtiles;
  }
  const int task = group * EE_REDUCE_TASKS + wave;
  if (group * EE_REDUCE_TASKS >= ntiles) return;      // whole workgroup
  const bool active = task < ntiles;
  const int m = mt * 16 + mc;
  float ss = 0.f;
  if (active) {
    EpiPre pre;
    epi_prefetch<EPI>(pre, out, task, row0 + m, m < M, lane);
    float sc[1] = {out.nin.inv_rms ? out.nin.inv_rms[min(m, M - 1)] : 1.0f};
    const bool sums = !out.nin.inv_rms && out.nin.ssq;
    NormPartials<1> part;
    if (sums) norm_request<1>(part, out.nin, row0 + mt * 16, 1, 1, 0, lane);
    f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
    const f32x4* pp = (const f32x4*)partial + ((size_t)task * TMT + mt) * 64 + lane;
    for (int s0 = 0; s0 < ksplit; s0 += 8) {
      f32x4 t[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) t[i] = __builtin_nontemporal_load(pp + (size_t)min(s0 + i, ksplit - 1) * ntiles * TMT * 64);
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if (s0 + i < ksplit) acc += t[i];
    }
    if (sums) norm_factors<1>(sc, part, out.nin, row0 + mt * 16, 1, 1, lane);
    epi_apply<EPI>(acc, sc[0], pre, out, task, row0 + m, m < M, N, lane, &ss);
  }
  if (EPI == EPI_ADD && out.nout.xn) {
    if (lane < 16) ssq[wave][lane] = ss;
    __syncthreads();
    if (threadIdx.x < 16)
      out.nout.ssq[(size_t)group * out.nout.stride + row0 + mt * 16 + threadIdx.x] =
          (ssq[0][threadIdx.x] + ssq[1][threadIdx.x]) + (ssq[2][threadIdx.x] + ssq[3][threadIdx.x]);
  }
}

size_t bf16_gemm_rows_scratch_floats(int ntiles, int ktiles) {
  const int ks = rows_ksplit(ntiles, ktiles);
  return ks > 1 ? (size_t)ks * ntiles * 32 * 256 : 0;       // [k share][weight tile][up to 32 row tiles][64 lanes x 4]
}

// plain launch, or with the offered timing events attached to the dispatch
template <typename K, typename... Args>
static void launch_timed(LaunchEvents* ev, K kernel, dim3 grid, dim3 blk, hipStream_t st, Args... args) {
  if (ev) {
    hipExtLaunchKernelGGL(kernel, grid, blk, 0, st, ev->start, ev->stop, 0, args...);
    ev->used = true;
  } else {
    hipLaunchKernelGGL(kernel, grid, blk, 0, st, args...);
  }
}

// returns whether the K shares took a reduction pass
template <int TMT>
static bool launch_gemm_rows(hipStream_t st, int epi, const uint4* W, int ntiles, int ktiles, const uint4* A, int row0, int M, int N,
                             const GemmOut& out, float* scratch) {
  const int ks = rows_ksplit(ntiles, ktiles), per = ceil_div(ktiles, ks);
  dim3 grid(ceil_div(ntiles, 2 * EE_ROWS_TN), ceil_div(ktiles, per)), blk(512), rblk(64 * EE_REDUCE_TASKS);
  const int ksr = grid.y;
  // every row tile holds rows; with 32 row tiles the kernel has no register to spare for the other variant
  const bool full = M > TMT * 16 - 16 || TMT == 32;
  // timing events are taken when this one kernel is the whole call (no K shares, hence no reduction pass)
  LaunchEvents* ev = ksr == 1 ? g_launch_events : nullptr;
  if (ev) g_launch_events = nullptr;
#define ROWS_LAUNCH(E_)                                                                                                          \
  do {                                                                                                                           \
    if (full) launch_timed(ev, gemm_rows_kernel<TMT, E_, true, EE_ROWS_TN>, grid, blk, st, W, ktiles, ntiles, A, row0, M, N, out, per, scratch); \
    else launch_timed(ev, gemm_rows_kernel<TMT, E_, TMT == 32, EE_ROWS_TN>, grid, blk, st, W, ktiles, ntiles, A, row0, M, N, out, per, scratch); \
  } while (0)
  // Seven weight tiles a workgroup where that deals a wide matrix more evenly over several rounds of workgroups: 70B gate/up at
  // 36 / 64 / 96 rows 153 / 159 / 176 us with eight, 148 / 152 / 169 with seven.  Not in one round (8B 43.5 either way at 36 rows,
  // 48.0 / 49.6 at 128) and not beyond 96 rows (70B at 144 rows 193 / 200), where the k-tile step, not the bytes, sets the time.
  if constexpr (TMT <= 8) {
    if (epi == EPI_SWIGLU && M <= 96 && grid.x > 256 && strip_load(ntiles, 7) < strip_load(ntiles, 8)) {
      grid.x = ceil_div(ntiles, 7);
      constexpr bool kFull = TMT == 4;      // (96 rows never fill eight row tiles)
      if (full && kFull) launch_timed(ev, gemm_rows_kernel<TMT, EPI_SWIGLU, kFull, EE_ROWS_TN, 7>, grid, blk, st, W, ktiles, ntiles, A, row0, M, N, out, per, scratch);
      else launch_timed(ev, gemm_rows_kernel<TMT, EPI_SWIGLU, false, EE_ROWS_TN, 7>, grid, blk, st, W, ktiles, ntiles, A, row0, M, N, out, per, scratch);
      return false;
    }
  }
  switch (epi) {
    case EPI_ADD: ROWS_LAUNCH(EPI_ADD); break;
    case EPI_SWIGLU: ROWS_LAUNCH(EPI_SWIGLU); break;
    case EPI_ROPE: ROWS_LAUNCH(EPI_ROPE); break;
    default: ROWS_LAUNCH(EPI_ARGMAX); break;
  }
#undef ROWS_LAUNCH
  if (ksr > 1) {
    dim3 rgrid(ceil_div(grid.x, 8) * 8 * (2 * EE_ROWS_TN / EE_REDUCE_TASKS) * ceil_div(M, 16));
    switch (epi) {
      case EPI_ADD: hipLaunchKernelGGL((gemm_rows_reduce_kernel<EPI_ADD>), rgrid, rblk, 0, st, scratch, ksr, ntiles, TMT, row0, M, N, out); break;
      case EPI_SWIGLU: hipLaunchKernelGGL((gemm_rows_reduce_kernel<EPI_SWIGLU>), rgrid, rblk, 0, st, scratch, ksr, ntiles, TMT, row0, M, N, out); break;
      case EPI_ROPE: hipLaunchKernelGGL((gemm_rows_reduce_kernel<EPI_ROPE>), rgrid, rblk, 0, st, scratch, ksr, ntiles, TMT, row0, M, N, out); break;
      default: hipLaunchKernelGGL((gemm_rows_reduce_kernel<EPI_ARGMAX>), rgrid, rblk, 0, st, scratch, ksr, ntiles, TMT, row0, M, N, out); break;
    }
  }
  return ksr > 1;
}

// Narrow matrices (few workgroup columns) without K shares: four weight tiles per workgroup and the rows cut into
// blocks of TMT*16 (grid.z), so that columns x blocks fill the chip and no partial tiles go through memory.
// Only the epilogues of the narrow projections are instantiated (O, down, adapters: residual add; QKV: RoPE).
template <int TMT, int TN>
static bool launch_gemm_rows_blocks(hipStream_t st, int epi, const uint4* W, int ntiles, int ktiles, const uint4* A, int row0, int M,
                                    int N, const GemmOut& out) {
  if (epi != EPI_ADD && epi != EPI_ROPE) return false;
  dim3 grid(ceil_div(ntiles, 2 * TN), 1, ceil_div(M, TMT * 16)), blk(512);
  const bool full = M % (TMT * 16) == 0;
  LaunchEvents* ev = g_launch_events;
  g_launch_events = nullptr;
#define ROWS_LAUNCH(E_)                                                                                                          \
  do {                                                                                                                           \
    if (full) launch_timed(ev, gemm_rows_kernel<TMT, E_, true, TN>, grid, blk, st, W, ktiles, ntiles, A, row0, M, N, out, ktiles, (float*)nullptr); \
    else launch_timed(ev, gemm_rows_kernel<TMT, E_, false, TN>, grid, blk, st, W, ktiles, ntiles, A, row0, M, N, out, ktiles, (float*)nullptr);    \
  } while (0)
  if (epi == EPI_ADD) ROWS_LAUNCH(EPI_ADD);
  else ROWS_LAUNCH(EPI_ROPE);
#undef ROWS_LAUNCH
  return true;
}

// Form of a blocked call: a pure function of the sizes (block_form), remembered for the last few.
static const BlockForm& choose_block(int epi, int ntiles, int ktiles, int M) {
  struct Memo { int ntiles, ktiles, M, kind; const BlockForm* form; };
  static thread_local Memo memo[8] = {};
  static thread_local unsigned next = 0;
  if (epi == EPI_ARGMAX) return kWideForms[0];
  const int kind = epi == EPI_SWIGLU ? 1 : 2;
  for (const Memo& m : memo)
    if (m.kind == kind && m.ntiles == ntiles && m.ktiles == ktiles && m.M == M) return *m.form;
  const BlockForm& best = block_form(kind == 1, ntiles, ktiles, M);
  memo[next++ & 7] = Memo{ntiles, ktiles, M, kind, &best};
  return best;
}
// the form that the test hook names (weight tiles + 100 * row tiles, 16 of them if unnamed), as far as this epilogue is built with it
static const BlockForm& forced_block(int epi, int tiles) {
  const int wt = tiles % 100, rt = tiles >= 100 ? tiles / 100 : 16;
  if (epi == EPI_ARGMAX) return kWideForms[0];
  if (epi == EPI_SWIGLU) return kWideForms[wt == 16 ? 0 : 1];
  for (const BlockForm& f : kNarrowForms)
    if (f.wt == wt && f.rt == rt) return f;
  return kNarrowForms[0];
}

template <int EPI, int TN, int TMT>
static void launch_block(hipStream_t st, const uint4* W, int ntiles, int ktiles, const uint4* A, int row0, int M, int N, const GemmOut& out) {
  const BlockOrder order = block_order(ntiles, M, 2 * TN, TMT);
  dim3 grid(8 * order.share), blk(512);
  LaunchEvents* ev = g_launch_events;
  g_launch_events = nullptr;
  launch_timed(ev, gemm_block_kernel<EPI, TN, TMT>, grid, blk, st, W, ktiles, ntiles, A, row0, M, N, out, order);
}
int g_rows_wide = 1;               // test and tuning hook: 0 keeps wide matrices in passes of up to 512 rows
int g_block_tiles = 0;             // test hook: > 0 runs every call that reaches bf16_gemm_rows blocked, in that form (forced_block)

// Form of the launch above for a call of M rows: row tiles per block, plus 100 with eight weight tiles per workgroup
// (TN = 4) instead of four; 0: use the K-share kernel (wide matrices, and shapes where it measured faster).
LaunchEvents* g_launch_events = nullptr;
int g_rows_blocks_override = -1;   // test and tuning hook: >= 0 replaces the choice below
int g_attn_pages_override = 0;
int g_attn_form = -1;              // test hook: >= 0 forces that attention kernel (ATTN_*) on every call
static int rows_blocks_form(int ntiles, int ktiles, int M) {
  if (g_rows_blocks_override >= 0) return g_rows_blocks_override;
  // measured on the 8B shapes (N 4096 and 6144): the blocks win for K <= 4096 from about 200 rows when columns x
  // blocks fit one round of workgroups; with K 14336 the K shares win at every row count.  Among the forms that
  // fit, the one with the cheapest k-tile step per workgroup (request time + MFMA time, in clocks) is taken.
  if (rows_ksplit(ntiles, ktiles) == 1 || ktiles > 128 || M <= 192) return 0;
  static const int forms[5][3] = {{2, 4, 192}, {2, 8, 320}, {4, 4, 320}, {4, 8, 512}, {2, 16, 576}};   // TN, TMT, clocks
  for (const auto& f : forms)
    if (ceil_div(ntiles, 2 * f[0]) * ceil_div(M, 16 * f[1]) <= 256) return (f[0] == 4 ? 100 : 0) + f[1];
  return 0;
}

// Whether a call of M rows runs as blocked launches over all its rows, else in parts of 512 rows and the rest.
//   wide matrices of 1536 and more weight tiles: from 257 rows (the row-tiled kernel needs two row blocks there, and measured
//     slower); not where a third row block of up to 128 rows would cost most of a second round of workgroups (8B gate/up at
//     520 / 608 / 640 rows: 164 / 169 / 170 us blocked, 146 / 150 / 154 as 512 rows and the rest; the 70B one, whose blocks
//     fill more than two rounds anyway, 488 blocked, 542 in parts)
//   narrow ones: see blocks_serve_narrow
// The hooks that force another form keep the parts.
static bool runs_blocked(bool wide, int ntiles, int ktiles, int M) {
  if (g_block_tiles > 0) return true;
  if (wide) return g_rows_wide && M > 256 && ntiles >= 1536 && !(M > 512 && M <= 640 && 3 * ceil_div(ntiles, 16) <= 512);
  if (M <= 512 || g_rows_blocks_override >= 0) return false;
  return blocks_serve_narrow(ntiles, ktiles, M);
}

bool bf16_takes_strips(int ntiles, int ktiles, int M) {
  const bool forced = (g_block_tiles > 0 || g_rows_blocks_override >= 0) && M > 16 && strips_large(ntiles, ktiles);
  return strips_serve(ntiles, ktiles, M) && !forced;
}

// more than 16 rows from row 0 of the operand; returns how many partial sums of squares per row an EPI_ADD call left
int bf16_gemm_rows(hipStream_t st, int epi, const bf16_t* W, int ntiles, int ktiles, const bf16_t* A, int M, int N,
                    const GemmOut& out0, float* scratch, float* inv_rms, int inv_cap) {
  const uint4* Wc = (const uint4*)W;
  const uint4* Ac = (const uint4*)A;
  const bool wide = epi == EPI_SWIGLU || epi == EPI_ARGMAX;
  const bool whole = runs_blocked(wide, ntiles, ktiles, M);
  // parts: blocked as many rows as inv_rms has factors for; else 512 rows and the rest, each streaming the weights once (three
  // parts of 400 rows cost what three of 512 do: gate/up of 1376 weight tiles at 1200 rows 417 us, 368 as 512 + 512 + 176)
  const int blk = whole ? ceil_div(ceil_div(M, ceil_div(M, max(512, inv_cap))), 16) * 16 : 512;
  if (M > blk) g_launch_events = nullptr;           // several launches: the caller's bracket times the call
  int parts_left = ntiles;                          // (EPI_ADD: all parts of a call take the same form)
  for (int m0 = 0; m0 < M; m0 += blk) {
    const int mc = min(blk, M - m0);
    const bool blocked = whole || (wide && runs_blocked(wide, ntiles, ktiles, mc));
    GemmOut out = out0;
    // Deferred norm factors: up to 192 rows every consumer sums the few partials of its own rows (see gemm_rows_reduce_kernel);
    // beyond, too many workgroups would each read too many, and one launch reduces them to factors.  The blocked kernel reads
    // factors only, and a part of a blocked call may be as short as one row
    if (out.nin.ssq && (mc > 192 || blocked)) {
      hipLaunchKernelGGL(norm_factor_kernel, dim3(ceil_div(mc, EE_NORM_ROWS)), dim3(1024), 0, st, out.nin.ssq + m0, out.nin.n_part, out.nin.stride,
                         out.nin.inv_d, out.nin.eps, inv_rms, mc);
      out.nin.inv_rms = inv_rms;
    }
    if (blocked) {
      const BlockForm& f = g_block_tiles > 0 ? forced_block(epi, g_block_tiles) : choose_block(epi, ntiles, ktiles, mc);
#define BLOCK_LAUNCH(E_, TN_, TMT_) launch_block<E_, TN_, TMT_>(st, Wc, ntiles, ktiles, Ac, m0, mc, N, out)
#define BLOCK_NARROW(E_)                                        \
  do {                                                          \
    if (f.rt == 8) BLOCK_LAUNCH(E_, 4, 8);                      \
    else if (f.rt == 12 && f.wt == 8) BLOCK_LAUNCH(E_, 4, 12);  \
    else if (f.rt == 12) BLOCK_LAUNCH(E_, 6, 12);               \
    else if (f.wt == 8) BLOCK_LAUNCH(E_, 4, 16);                \
    else if (f.wt == 12) BLOCK_LAUNCH(E_, 6, 16);               \
    else BLOCK_LAUNCH(E_, 8, 16);                               \
  } while (0)
      switch (epi) {
        case EPI_ARGMAX: BLOCK_LAUNCH(EPI_ARGMAX, 8, 16); break;
        case EPI_SWIGLU: if (f.wt == 16) BLOCK_LAUNCH(EPI_SWIGLU, 8, 16); else BLOCK_LAUNCH(EPI_SWIGLU, 6, 16); break;
        case EPI_ROPE: BLOCK_NARROW(EPI_ROPE); break;
        default: BLOCK_NARROW(EPI_ADD); break;
      }
#undef BLOCK_NARROW
#undef BLOCK_LAUNCH
      continue;
    }
    const int bt = rows_blocks_form(ntiles, ktiles, epi == EPI_ADD ? min(M, blk) : mc);
    if (m0 > 0 && bf16_takes_strips(ntiles, ktiles, mc) && (epi != EPI_ADD || bt > 0 || rows_ksplit(ntiles, ktiles) == 1)) {
      bf16_gemm(st, epi, W, ntiles, ktiles, A, mc, N, out, m0);        // (as such a call by itself; leaves a partial sum per weight tile)
      continue;
    }
    if (bt == 4 && launch_gemm_rows_blocks<4, 2>(st, epi, Wc, ntiles, ktiles, Ac, m0, mc, N, out)) continue;
    if (bt == 8 && launch_gemm_rows_blocks<8, 2>(st, epi, Wc, ntiles, ktiles, Ac, m0, mc, N, out)) continue;
    if (bt == 16 && launch_gemm_rows_blocks<16, 2>(st, epi, Wc, ntiles, ktiles, Ac, m0, mc, N, out)) continue;
    if (bt == 104 && launch_gemm_rows_blocks<4, 4>(st, epi, Wc, ntiles, ktiles, Ac, m0, mc, N, out)) continue;
    if (bt == 108 && launch_gemm_rows_blocks<8, 4>(st, epi, Wc, ntiles, ktiles, Ac, m0, mc, N, out)) continue;
    bool reduced;
    if (mc <= 64) reduced = launch_gemm_rows<4>(st, epi, Wc, ntiles, ktiles, Ac, m0, mc, N, out, scratch);
    else if (mc <= 128) reduced = launch_gemm_rows<8>(st, epi, Wc, ntiles, ktiles, Ac, m0, mc, N, out, scratch);
    else if (mc <= 192) reduced = launch_gemm_rows<12>(st, epi, Wc, ntiles, ktiles, Ac, m0, mc, N, out, scratch);
    else if (mc <= 256) reduced = launch_gemm_rows<16>(st, epi, Wc, ntiles, ktiles, Ac, m0, mc, N, out, scratch);
    else if (mc <= 384) reduced = launch_gemm_rows<24>(st, epi, Wc, ntiles, ktiles, Ac, m0, mc, N, out, scratch);
    else reduced = launch_gemm_rows<32>(st, epi, Wc, ntiles, ktiles, Ac, m0, mc, N, out, scratch);
    if (reduced) parts_left = ceil_div(ntiles, EE_REDUCE_TASKS);
  }
  return parts_left;
}

// QKV in whole strips and a half a workgroup (see strips_half)
template <int MT, int NS, int U>
static void launch_gemm_half(hipStream_t st, const uint4* W, int ntiles, int ktiles, const uint4* A, int row0, int M, int N, const GemmOut& out, int ksplit) {
  LaunchEvents* ev = g_launch_events;
  g_launch_events = nullptr;
  launch_timed(ev, gemm_skinny_kernel<MT, EPI_ROPE, NS, U, true>, dim3(half_grid(ntiles, NS)), dim3(64 * ksplit), st, W, ktiles, ntiles,
               A, row0, M, N, out, ksplit);
}

template <int MT, int NS, int U>
static void launch_gemm_mt(hipStream_t st, int epi, const uint4* W, int ntiles, int ktiles, const uint4* A, int row0, int M, int N,
                           const GemmOut& out, int nw, int ksplit) {
  dim3 blk(64 * nw), grid(ceil_div(ntiles, nw / ksplit * NS));
  LaunchEvents* ev = g_launch_events;
  g_launch_events = nullptr;                       // one launch per offer
#define SKINNY_LAUNCH(E_) launch_timed(ev, gemm_skinny_kernel<MT, E_, NS, U>, grid, blk, st, W, ktiles, ntiles, A, row0, M, N, out, ksplit)
  switch (epi) {
    case EPI_ADD: SKINNY_LAUNCH(EPI_ADD); break;
    case EPI_SWIGLU: SKINNY_LAUNCH(EPI_SWIGLU); break;
    case EPI_ROPE: SKINNY_LAUNCH(EPI_ROPE); break;
    default: SKINNY_LAUNCH(EPI_ARGMAX); break;
  }
#undef SKINNY_LAUNCH
}

void bf16_gemm(hipStream_t st, int epi, const bf16_t* W, int ntiles, int ktiles, const bf16_t* A, int M, int N, const GemmOut& out, int row0) {
  const uint4* Wc = (const uint4*)W;
  const uint4* Ac = (const uint4*)A;
  const StripShape sh = strip_shape(ntiles, ktiles, M);
  if (const int ns = epi == EPI_ROPE ? strips_half(ntiles, ktiles, M) : 0) {
    if (ns == 3) launch_gemm_half<1, 3, 4>(st, Wc, ntiles, ktiles, Ac, row0, M, N, out, sh.ksplit);
    else launch_gemm_half<1, 2, 4>(st, Wc, ntiles, ktiles, Ac, row0, M, N, out, sh.ksplit);
    return;
  }
#define STRIPS(MT_, NS_, U_) launch_gemm_mt<MT_, NS_, U_>(st, epi, Wc, ntiles, ktiles, Ac, row0, M, N, out, sh.nw, sh.ksplit)
  if (M <= 16) {
    if (sh.ns == 4) STRIPS(1, 4, 4);
    else if (sh.ns == 2) STRIPS(1, 2, 4);
    else STRIPS(1, 1, 8);
  } else {
    if (sh.ns == 7) STRIPS(2, 7, 1);
    else if (sh.ns == 4) STRIPS(2, 4, 2);
    else if (sh.ns == 2) STRIPS(2, 2, 4);
    else STRIPS(2, 1, 4);
  }
#undef STRIPS
}

// one workgroup of 1024 threads per row; the row's partials lie side by side ([row][tile]), so a wave's load is one
// contiguous 256 bytes; eight independent partials per thread are requested at once
__global__ __launch_bounds__(1024) void bf16_argmax_reduce_kernel(const float* __restrict__ pmax, const int* __restrict__ pidx,
                                                                   int ntiles, int pstride, int* v, TakeToken take) {
  __shared__ float bv[16];
  __shared__ int bi[16];
  const int m = blockIdx.x;
  float best = -INFINITY; int idx = 0x7fffffff;
  for (int t0 = threadIdx.x; t0 < ntiles; t0 += 8 * 1024) {
    float x[8]; int xi[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int t = min(t0 + j * 1024, ntiles - 1);
      x[j] = pmax[(size_t)m * pstride + t]; xi[j] = pidx[(size_t)m * pstride + t];
    }
#pragma unroll
    for (int j = 0; j < 8; ++j)      // a clamped duplicate carries the same (value, index): harmless
      if (x[j] > best || (x[j] == best && xi[j] < idx)) { best = x[j]; idx = xi[j]; }
  }
  // within the wave by shuffles, then the sixteen waves' results through LDS (one barrier)
  for (int sh = 32; sh > 0; sh >>= 1) {
    const float o = __shfl_xor(best, sh, 64); const int oi = __shfl_xor(idx, sh, 64);
    if (o > best || (o == best && oi < idx)) { best = o; idx = oi; }
  }
  if ((threadIdx.x & 63) == 0) { bv[threadIdx.x >> 6] = best; bi[threadIdx.x >> 6] = idx; }
  __syncthreads();
  if (threadIdx.x < 64) {
    best = threadIdx.x < 16 ? bv[threadIdx.x] : -INFINITY; idx = threadIdx.x < 16 ? bi[threadIdx.x] : 0x7fffffff;
    for (int sh = 8; sh > 0; sh >>= 1) {
      const float o = __shfl_xor(best, sh, 64); const int oi = __shfl_xor(idx, sh, 64);
      if (o > best || (o == best && oi < idx)) { best = o; idx = oi; }
    }
    if (threadIdx.x == 0) { v[m] = idx; take_token(take, m, idx); }
  }
}
void bf16_argmax_reduce(hipStream_t st, const float* pmax, const int* pidx, int ntiles, int pstride, int M, int* v, const TakeToken& take) {
  hipLaunchKernelGGL(bf16_argmax_reduce_kernel, dim3(M), dim3(1024), 0, st, pmax, pidx, ntiles, pstride, v, take);
}

// ---------------------------------------------------------------------------------------------
// k-query causal-in-block GQA attention over the paged cache, split over the KV axis.
// A sequence's block of m rows times the `rep` query heads sharing one KV head forms nq = m*rep
// query rows, cut into 16-row q-tiles.  Workgroup = (KV split, KV head [x group of q-tiles],
// sequence), eight waves with fixed roles: six compute waves, each owning one q-tile, and two loader
// waves.  The split's pages stream HBM -> loader registers -> LDS: each loader fetches half of every
// page (1 KiB chunks) and keeps three pages in flight in its registers, which is what hides HBM latency;
// the compute waves read whole pages back from a three-slot LDS ring, so a page crosses HBM, L2 and the
// vector memory path once however many q-tiles consume it.  One barrier per page hands a slot over.  Per page (64 positions) and q-tile:
//   S^T[pos][q] = K[pos][:] . Q[q][:]        4 pos-tiles x D/32 MFMAs  (K page = A operand, Q^T = B)
//   online softmax per q column (= per lane%16; the 4 lane groups hold 16 positions each)
//   O^T[d][q] += V^T[d][pos] P^T[pos][q]     D/16 d-tiles x 2 MFMAs    (V page = A operand, P^T = B)
// The page's element order (common.h) makes the S^T accumulators, once exponentiated and packed to
// bf16, exactly the B operand of the second product: no shuffles beyond the row statistics.
// Row r of the block sits at position p0+r and may see cache positions 0..p0+r (its own block rows
// included, they were appended just before).  Dead cache entries (>= p0+m) are never trusted:
// scores are masked by select and V elements are zeroed, so NaN there cannot leak.
// With one split the normalised output goes straight to the O-projection operand; otherwise the
// partials (max, sum, unnormalised O) go to scratch and attn_merge_kernel combines them.
// ---------------------------------------------------------------------------------------------
// maximum over the four 16-lane rows of a wave, delivered to every lane: lane l ends up with
// max(x[l % 16 + 16 r], r = 0..3).  v_permlane16_swap exchanges the odd rows of its first operand with the
// even rows of its second, v_permlane32_swap the upper half of the first with the lower half of the second.
__device__ inline float colmax4(float x) {
  typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));
  u32x2_t r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

#define EE_MAX_SPLITS 64
#define EE_ATTN_WAVES 8
#define EE_ATTN_COMPUTE 6   // compute waves = q-tiles per workgroup; the other waves load
#define EE_ATTN_AHEAD 3     // pages each loader wave keeps in flight

template <int D, int QPW>
__global__ __launch_bounds__(64 * EE_ATTN_WAVES) void attn_kernel(const uint4* __restrict__ Q, const bf16_t* __restrict__ kv,
                                                                  const int* seq_m, const int* seq_p0, const int* seq_qt0,
                                                                  const int* seq_row0, const int* block_table, int pos_add, int rep,
                                                                  int total_qt, int Hkv, int layer, int n_pages, int pps, int nsplit,
                                                                  int per, float* part_o, float* part_ml, bf16_t* __restrict__ out,
                                                                  int out_ktiles) {
  constexpr int DS = D / 32, DT = D / 16;
  constexpr int KCH = 4 * DS, CH = KCH + 2 * DT;       // 1 KiB chunks of a page: K first, then V
  constexpr int NL = EE_ATTN_WAVES - EE_ATTN_COMPUTE, PF = EE_ATTN_AHEAD;
  constexpr int CPL = CH / NL;                         // chunks each loader wave fetches per page
  static_assert(CH % NL == 0, "page chunks must divide among the loader waves");
  __shared__ u32x4 lds[3][CH * 64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, g = lane >> 4, qc = lane & 15;
  const int b = blockIdx.z, kvh = blockIdx.y % Hkv, sp = blockIdx.x;
  const int pg0 = sp * per;                            // every split takes `per` pages: a short sequence has fewer splits
  const int* bt = block_table + b * pps;
  // every scalar the workgroup needs before its first KV fetch is requested ahead of the first branch,
  // so the prologue costs one memory round trip, not one per dependent step (indices clamped into the table)
  int m = seq_m[b], sp0 = seq_p0[b], sqt0 = seq_qt0[b];
  int bt0[EE_ATTN_AHEAD];
#pragma unroll
  for (int q = 0; q < EE_ATTN_AHEAD; ++q) bt0[q] = bt[min(pg0 + q, pps - 1)];
  static_assert(EE_ATTN_AHEAD == 3, "the statement below names the look-ahead entries one by one");
  // ties the values together ahead of the branches (not volatile and without a memory clobber, so later
  // table lookups stay scalar loads)
  asm("" : "+s"(m), "+s"(sp0), "+s"(sqt0), "+s"(bt0[0]), "+s"(bt0[1]), "+s"(bt0[2]));
  if (m == 0) return;                                  // whole workgroup
  const int nq = m * rep;
  const int qt0 = (blockIdx.y / Hkv) * (EE_ATTN_COMPUTE * QPW);
  if (qt0 * 16 >= nq) return;                          // whole workgroup
  const int p0 = sp0 + pos_add, kv_end = p0 + m;
  const int npages = (kv_end + EE_PAGE - 1) / EE_PAGE;
  const int pg1 = min(npages, pg0 + per);
  if (pg0 >= npages) return;                           // whole workgroup; the merge pass knows this sequence's split count

  const bool loader = wave >= EE_ATTN_COMPUTE;
  const int lw = wave - EE_ATTN_COMPUTE;
  int limit[QPW];
  bool has[QPW];
  u32x4 qf[QPW][DS];
  float mrun[QPW];
  f32x4 o[QPW][DT], lacc[QPW];   // lacc: running row sums (every element of a lane holds its column's sum)
#pragma unroll
  for (int i = 0; i < QPW; ++i) {
    const int qt = qt0 + wave * QPW + i;
    has[i] = !loader && qt * 16 < nq;
    const int qrow = qt * 16 + qc;
    limit[i] = (has[i] && qrow < nq) ? p0 + qrow / rep : -1;
    const int gqt = sqt0 + (has[i] ? qt : 0);
#pragma unroll
    for (int s = 0; s < DS; ++s) qf[i][s] = ((const u32x4*)Q)[(((size_t)kvh * total_qt + gqt) * DS + s) * 64 + lane];
    mrun[i] = -INFINITY; lacc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) o[i][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  // loader side: st[q] holds this wave's chunks (lw, lw + NL, ...) of the page q pages ahead (mod PF)
  u32x4 st[PF][CPL];
#define ATTN_FETCH(q_, page_)                                                                                \
  do {                                                                                                       \
    const u32x4* src_ = (const u32x4*)(kv + kv_slab(layer, page_, kvh, n_pages, Hkv, D)) + lw * 64 + lane;   \
    _Pragma("unroll") for (int j = 0; j < CPL; ++j) st[q_][j] = __builtin_nontemporal_load(src_ + j * NL * 64); \
  } while (0)
#define ATTN_DEPOSIT(buf_, q_)                                                                               \
  do {                                                                                                       \
    u32x4* dst_ = lds[buf_] + lw * 64 + lane;                                                                \
    _Pragma("unroll") for (int j = 0; j < CPL; ++j) dst_[j * NL * 64] = st[q_][j];                           \
  } while (0)
  // Scores are kept in base-2 units (s * log2(e)/sqrt(D)) so that the exponential is a bare v_exp_f32;
  // the row sums of the bf16-rounded weights come from one more MFMA column block (an all-ones A
  // operand), not from the vector ALU.  One step handles the scores and softmax of page pg and the
  // P.V product of page pg-1, whose weights the previous step left in registers: the two are
  // independent, so the second's MFMAs run under the first's vector arithmetic.  TAIL steps (a page
  // reaching into the block or past the end) mask scores and zero dead V.
  const float sc2 = 1.4426950408889634f / sqrtf((float)D);
  const u32x4 ones = {0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u};
  u32x4 Pp0 = {0u, 0u, 0u, 0u}, Pp1 = {0u, 0u, 0u, 0u};   // weights of the previous page (B operand of P.V)
  // LDS fragment reads are issued as whole groups ahead of the MFMAs that consume them, and scheduling
  // barriers keep the compiler from sinking them back next to their uses (which would expose the LDS
  // latency once per fragment).
  auto pv_mfma = [&](auto tail_c, const u32x4 (&vf)[2 * DT], int ppg) __attribute__((always_inline)) {
    constexpr bool TAIL = decltype(tail_c)::value;
    const int pbase = ppg * EE_PAGE + 16 * g;
    lacc[0] = mfma16(ones, Pp0, lacc[0]);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {     // the two MFMAs of a d-tile depend on each other: keep them 8 apart
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        u32x4 v = vf[dt * 2 + ks];
        if (TAIL) {   // zero V at dead positions: element j of the fragment is position pbase + 8*ks + j
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const int pa = pbase + 8 * ks + 2 * j;
            v[j] &= pa + 1 < kv_end ? 0xffffffffu : (pa < kv_end ? 0xffffu : 0u);
          }
        }
        o[0][dt] = mfma16(v, ks == 0 ? Pp0 : Pp1, o[0][dt]);
      }
    }
    lacc[0] = mfma16(ones, Pp1, lacc[0]);
  };
  auto step = [&](auto tail_c, auto prev_c, int slot, int pslot, int pg) __attribute__((always_inline)) {
    constexpr bool TAIL = decltype(tail_c)::value, PREV = decltype(prev_c)::value;
    const u32x4* L = &lds[0][0] + slot * (CH * 64) + lane;     // the slot is a run-time value: one loop body serves the whole ring
    const u32x4* Lp = &lds[0][0] + pslot * (CH * 64) + lane;
    const int base = pg * EE_PAGE + 16 * g;          // this lane group holds positions base .. base+15
    u32x4 kf[4 * DS];
#pragma unroll
    for (int c = 0; c < 4 * DS; ++c) kf[c] = L[c * 64];
    __builtin_amdgcn_sched_barrier(0);
    f32x4 s4[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) s4[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < DS; ++s)
#pragma unroll
      for (int t = 0; t < 4; ++t) s4[t] = mfma16(kf[t * DS + s], qf[0][s], s4[t]);
    u32x4 vf[2 * DT];
    if (PREV) {
#pragma unroll
      for (int c = 0; c < 2 * DT; ++c) vf[c] = Lp[(KCH + c) * 64];
    }
    __builtin_amdgcn_sched_barrier(0);
    if (PREV) pv_mfma(tail_c, vf, pg - 1);
    // raw scores; the maximum is taken before scaling (the scale is positive) and the scale is folded
    // into the exponent's argument as one fused multiply-add
    float tmax = -INFINITY;
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        if (TAIL && base + 4 * t + v > limit[0]) s4[t][v] = -INFINITY;
        tmax = fmaxf(tmax, s4[t][v]);
      }
    tmax *= sc2;
    // running maximum of the column, shared by the four lane groups that hold its positions (two
    // register swaps across lane rows, no LDS traffic).  Everything up to the packed weights is
    // straight-line code, so the exponentials can be scheduled under the MFMAs; only the rescaling of
    // the accumulators, which is rare once the maximum has settled, sits behind a branch at the end.
    tmax = colmax4(tmax);
    const float mnew = fmaxf(mrun[0], tmax);
    const float msafe = mnew == -INFINITY ? 0.f : mnew;
    const float alpha = __builtin_amdgcn_exp2f(mrun[0] - msafe);
    mrun[0] = mnew;
    const float nm = -msafe;
    uint32_t pk[8];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      pk[2 * t] = pack2(__builtin_amdgcn_exp2f(fmaf(s4[t][0], sc2, nm)), __builtin_amdgcn_exp2f(fmaf(s4[t][1], sc2, nm)));
      pk[2 * t + 1] = pack2(__builtin_amdgcn_exp2f(fmaf(s4[t][2], sc2, nm)), __builtin_amdgcn_exp2f(fmaf(s4[t][3], sc2, nm)));
    }
    // (the empty statement pins the weights ahead of the branch: otherwise the exponentials are sunk
    // below it, out of the block that holds the MFMAs)
    asm volatile("" : "+v"(pk[0]), "+v"(pk[1]), "+v"(pk[2]), "+v"(pk[3]), "+v"(pk[4]), "+v"(pk[5]), "+v"(pk[6]), "+v"(pk[7]));
    if (__builtin_amdgcn_ballot_w64(alpha != 1.0f) != 0) {
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) { o[0][dt][0] *= alpha; o[0][dt][1] *= alpha; o[0][dt][2] *= alpha; o[0][dt][3] *= alpha; }
      lacc[0][0] *= alpha; lacc[0][1] *= alpha; lacc[0][2] *= alpha; lacc[0][3] *= alpha;
    }
    Pp0 = u32x4{pk[0], pk[1], pk[2], pk[3]};   // positions base+0..7  (pos-tiles 0, 1)
    Pp1 = u32x4{pk[4], pk[5], pk[6], pk[7]};   // positions base+8..15 (pos-tiles 2, 3)
  };
  auto pv_last = [&](auto tail_c, int pslot, int ppg) __attribute__((always_inline)) {
    const u32x4* Lp = &lds[0][0] + pslot * (CH * 64) + lane;
    u32x4 vf[2 * DT];
#pragma unroll
    for (int c = 0; c < 2 * DT; ++c) vf[c] = Lp[(KCH + c) * 64];
    pv_mfma(tail_c, vf, ppg);
  };
  // software pipeline over a ring of three LDS slots (slot = page offset mod 3): while the compute waves
  // work on page p (scores) and p-1 (P.V), the loaders drop page p+1 into the third slot and request
  // page p+1+PF; every wave passes one barrier per page
  // (the two roles run separate loops with the same number of barriers, so neither carries the other's
  // registers)
  if (loader) {
    // Loads return in order and the compiler places the waits from what it can prove about the order of
    // issue, so the long-split path is kept free of branches from the first fetch to the end of its
    // steady-state loop: one conditional fetch on the way in would make every deposit of the loop wait
    // for all outstanding loads.
    int pg = pg0;
    if (pg0 + 2 * PF < pg1) {
#pragma unroll
      for (int q = 0; q < PF; ++q) ATTN_FETCH(q, bt0[q]);
      ATTN_DEPOSIT(0, 0);
      ATTN_FETCH(0, bt[pg0 + PF]);
      __syncthreads();
      for (; pg + 2 * PF < pg1; pg += PF) {
#pragma unroll
        for (int u = 0; u < PF; ++u) {
          ATTN_DEPOSIT((u + 1) % 3, (u + 1) % PF);
          ATTN_FETCH((u + 1) % PF, bt[pg + u + 1 + PF]);
          __syncthreads();
        }
      }
    } else {
#pragma unroll
      for (int q = 0; q < PF; ++q)
        if (pg0 + q < pg1) ATTN_FETCH(q, bt0[q]);
      if (pg0 < pg1) ATTN_DEPOSIT(0, 0);
      if (pg0 + PF < pg1) ATTN_FETCH(0, bt[pg0 + PF]);
      __syncthreads();
    }
    for (; pg < pg1; pg += PF) {     // guarded tail (and short splits): one barrier per remaining page
#pragma unroll
      for (int u = 0; u < PF; ++u) {
        const int p = pg + u;
        if (p >= pg1) break;
        if (p + 1 < pg1) ATTN_DEPOSIT((u + 1) % 3, (u + 1) % PF);
        if (p + 1 + PF < pg1) ATTN_FETCH((u + 1) % PF, bt[p + 1 + PF]);
        __syncthreads();
      }
    }
    return;
  }
#undef ATTN_FETCH
#undef ATTN_DEPOSIT
  static_assert(PF == 3 && QPW == 1, "three ring slots, one q-tile per compute wave");
  // Compute side: 1 + (pg1 - pg0) barriers like the loaders.  The page loop is cut into three plain loops
  // (first page, pages wholly before the block, pages reaching into it) whose bodies are one step
  // variant each, so the accumulators stay in place: no variant merges inside the steady-state loop.
  __syncthreads();
  if (!has[0]) {
    for (int pg = pg0; pg < pg1; ++pg) __syncthreads();
    return;
  }
  {
    const int first_tail = p0 / EE_PAGE;       // pages from here on reach into the block or past the end
    int pg = pg0, slot = 0, pslot = 2;
    if (pg >= first_tail) step(std::true_type{}, std::false_type{}, slot, pslot, pg);
    else step(std::false_type{}, std::false_type{}, slot, pslot, pg);
    __syncthreads();
    pslot = 0; slot = 1; ++pg;
    const int pe = min(pg1, first_tail);
    for (; pg < pe; ++pg) {
      step(std::false_type{}, std::true_type{}, slot, pslot, pg);
      __syncthreads();
      pslot = slot; slot = slot == 2 ? 0 : slot + 1;
    }
    for (; pg < pg1; ++pg) {
      step(std::true_type{}, std::true_type{}, slot, pslot, pg);
      __syncthreads();
      pslot = slot; slot = slot == 2 ? 0 : slot + 1;
    }
    // P.V of the split's last page (its slot is not written again)
    if (pg1 > first_tail) pv_last(std::true_type{}, pslot, pg1 - 1);
    else pv_last(std::false_type{}, pslot, pg1 - 1);
  }

#pragma unroll
  for (int i = 0; i < QPW; ++i) {
    if (!has[i]) continue;
    const int qt = qt0 + wave * QPW + i, gqt = sqt0 + qt, qrow = qt * 16 + qc;
    const float l = lacc[i][0];
    if (nsplit == 1) {
      if (qrow < nq) {
        const float inv = 1.0f / l;
        const int row = seq_row0[b] + qrow / rep, col0 = (kvh * rep + qrow % rep) * D + 4 * g;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
          *(uint2*)(out + act_offset(row, col0 + dt * 16, out_ktiles)) =
              make_uint2(pack2(o[i][dt][0] * inv, o[i][dt][1] * inv), pack2(o[i][dt][2] * inv, o[i][dt][3] * inv));
      }
    } else {
      // partial O of a split: [d-tile][lane] float4, the accumulator registers as they are
      const size_t slot = ((size_t)gqt * Hkv + kvh) * nsplit + sp;
      if (g == 0) *(float2*)(part_ml + slot * 32 + qc * 2) = make_float2(mrun[i], l);
      float4* po = (float4*)part_o + slot * (DT * 64) + lane;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) po[dt * 64] = make_float4(o[i][dt][0], o[i][dt][1], o[i][dt][2], o[i][dt][3]);
    }
  }
}

// ---------------------------------------------------------------------------------------------
// The same attention for long blocks (context build): a workgroup takes 128 query rows (eight q-tiles) of one KV head.
// Wave (qg, par) owns q-tiles 2*qg and 2*qg+1 and every second page (page mod 2 == par): two q-tiles per wave halve the LDS
// reads per product (32 KiB of fragments serve 68 MFMAs; the kernel above, one q-tile per wave, is bound by those reads), and
// the two waves of a SIMD, one of each parity, run one's vector arithmetic under the other's MFMAs.  Pages reach LDS by direct
// global->LDS loads into two slots of two pages each; a step is one pair of pages, with one barrier, and requests the next
// pair while it works.  The two parities of a q-tile meet in LDS at the end.  Nothing is split over workgroups, so where this
// kernel runs a row's result depends on its own sequence alone (the batch decides whether it runs).  8B width: 2048 rows without a context 61-62 us a layer (136 in four 512-row passes of
// the kernel above), the 4096-row passes of an 8190-token prompt 385 us on average, 714 TFLOP/s (695 us).  A step of two pages
// takes about 6000 clocks against 2100-2400 each of MFMAs, vector arithmetic and LDS reads; the P.V product of the previous
// page under this page's softmax inside each wave, as in the kernel above, only lengthened it (411 us).  blockIdx.x is the KV
// head (with eight of them each XCD keeps one head's pages in its L2), the blocks with the most pages come first.
// ---------------------------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(512) void attn_block_kernel(const uint4* __restrict__ Q, const bf16_t* __restrict__ kv, const int* seq_m,
                                                         const int* seq_p0, const int* seq_qt0, const int* seq_row0,
                                                         const int* block_table, int pos_add, int rep, int total_qt, int Hkv, int layer,
                                                         int n_pages, int pps, bf16_t* __restrict__ out, int out_ktiles) {
  constexpr int DS = D / 32, DT = D / 16, KCH = 4 * DS, CH = KCH + 2 * DT;     // 1 KiB chunks of a page: K first, then V
  constexpr int CPW = CH / 4;                                                  // chunks a wave requests per step
  __shared__ u32x4 lds[4][CH * 64];                                            // slot 2 * (step mod 2) + parity
  __shared__ float2 ml[4][2][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, g = lane >> 4, qc = lane & 15;
  const int wave_s = __builtin_amdgcn_readfirstlane(wave), qg = wave_s & 3, par = wave_s >> 2;
  const int kvh = blockIdx.x, b = blockIdx.z, grp = gridDim.y - 1 - blockIdx.y;
  const int m = seq_m[b], nq = m * rep, qt0 = grp * 8;
  if (qt0 * 16 >= nq) return;                          // whole workgroup (also m == 0)
  const int p0 = seq_p0[b] + pos_add, kv_end = p0 + m, sqt0 = seq_qt0[b];
  const int tok0 = qt0 * 16 / rep, tok1 = min(m - 1, (qt0 * 16 + 127) / rep);  // first and last token of the block
  const int npg = (p0 + tok1) / EE_PAGE + 1, first_masked = (p0 + tok0 + 1) / EE_PAGE, nst = (npg + 1) >> 1;
  const int* bt = block_table + b * pps;
  typedef const __attribute__((address_space(1))) void* gptr_t;
  typedef __attribute__((address_space(3))) void* lptr_t;
  const unsigned lds0 = __builtin_amdgcn_readfirstlane((unsigned)(size_t)(lptr_t)&lds[0][0]);
  // this wave's share of a step: chunks qg*CPW .. of the page of its own parity
  auto request = [&](int step, int page) __attribute__((always_inline)) {
    const u32x4* src = (const u32x4*)(kv + kv_slab(layer, page, kvh, n_pages, Hkv, D)) + qg * CPW * 64 + lane;
    const unsigned dst = lds0 + 1024u * (((step & 1) * 2 + par) * CH + qg * CPW);
#pragma unroll
    for (int j = 0; j < CPW; ++j) __builtin_amdgcn_global_load_lds((gptr_t)(src + j * 64), (lptr_t)(size_t)(dst + 1024u * j), 16, 0, 0);
  };
  request(0, bt[min(par, npg - 1)]);
  int next_page = bt[min(2 + par, npg - 1)];
  bool has[2];
  int limit[2];
  u32x4 qf[2][DS];
  float mrun[2];
  f32x4 o[2][DT], lacc[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int qt = qt0 + 2 * qg + i, qrow = qt * 16 + qc;
    has[i] = qt * 16 < nq;
    limit[i] = qrow < nq ? p0 + qrow / rep : -1;
    const int gqt = sqt0 + (has[i] ? qt : qt0);
#pragma unroll
    for (int s = 0; s < DS; ++s) qf[i][s] = ((const u32x4*)Q)[(((size_t)kvh * total_qt + gqt) * DS + s) * 64 + lane];
    mrun[i] = -INFINITY; lacc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) o[i][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  const float sc2 = 1.4426950408889634f / sqrtf((float)D);         // scores in base-2 units, as above
  const u32x4 ones = {0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u};
  auto page_step = [&](auto masked_c, const u32x4* L, int pg) __attribute__((always_inline)) {
    constexpr bool MASKED = decltype(masked_c)::value;
    const int base = pg * EE_PAGE + 16 * g;            // this lane group holds positions base .. base+15
    f32x4 s4[2][4];
#pragma unroll
    for (int h = 0; h < 2; ++h) {                      // (fragments in halves: 256 registers hold no more)
      u32x4 kf[2 * DS];
#pragma unroll
      for (int c = 0; c < 2 * DS; ++c) kf[c] = L[(h * 2 * DS + c) * 64];
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int i = 0; i < 2; ++i) s4[i][2 * h + t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < DS; ++s)
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int i = 0; i < 2; ++i) s4[i][2 * h + t] = mfma16(kf[t * DS + s], qf[i][s], s4[i][2 * h + t]);
      __builtin_amdgcn_sched_barrier(0);
    }
    u32x4 vf[DT];                                      // first half of V, requested under the softmax
#pragma unroll
    for (int c = 0; c < DT; ++c) vf[c] = L[(KCH + c) * 64];
    u32x4 P[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      float tmax = -INFINITY;
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          if (MASKED && base + 4 * t + v > limit[i]) s4[i][t][v] = -INFINITY;
          tmax = fmaxf(tmax, s4[i][t][v]);
        }
      tmax = colmax4(tmax * sc2);
      const float mnew = fmaxf(mrun[i], tmax);
      const float msafe = mnew == -INFINITY ? 0.f : mnew;
      const float alpha = __builtin_amdgcn_exp2f(mrun[i] - msafe), nm = -msafe;
      mrun[i] = mnew;
      uint32_t pk[8];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        pk[2 * t] = pack2(__builtin_amdgcn_exp2f(fmaf(s4[i][t][0], sc2, nm)), __builtin_amdgcn_exp2f(fmaf(s4[i][t][1], sc2, nm)));
        pk[2 * t + 1] = pack2(__builtin_amdgcn_exp2f(fmaf(s4[i][t][2], sc2, nm)), __builtin_amdgcn_exp2f(fmaf(s4[i][t][3], sc2, nm)));
      }
      if (__builtin_amdgcn_ballot_w64(alpha != 1.0f) != 0) {       // (rare once the maximum has settled)
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) { o[i][dt][0] *= alpha; o[i][dt][1] *= alpha; o[i][dt][2] *= alpha; o[i][dt][3] *= alpha; }
        lacc[i][0] *= alpha; lacc[i][1] *= alpha; lacc[i][2] *= alpha; lacc[i][3] *= alpha;
      }
      P[i][0] = u32x4{pk[0], pk[1], pk[2], pk[3]};
      P[i][1] = u32x4{pk[4], pk[5], pk[6], pk[7]};
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      __builtin_amdgcn_sched_barrier(0);
      if (h) {
#pragma unroll
        for (int c = 0; c < DT; ++c) vf[c] = L[(KCH + DT + c) * 64];
      }
#pragma unroll
      for (int i = 0; i < 2; ++i) lacc[i] = mfma16(ones, P[i][h], lacc[i]);
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int dt = 0; dt < DT / 2; ++dt) {
          u32x4 v = vf[dt * 2 + ks];
          if (MASKED) {     // dead positions (>= kv_end) may hold anything: zero their V
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              const int pa = base + 8 * ks + 2 * j;
              v[j] &= pa + 1 < kv_end ? 0xffffffffu : (pa < kv_end ? 0xffffu : 0u);
            }
          }
#pragma unroll
          for (int i = 0; i < 2; ++i) o[i][h * DT / 2 + dt] = mfma16(v, P[i][ks], o[i][h * DT / 2 + dt]);
        }
    }
  };
  auto open_step = [&](int st) __attribute__((always_inline)) {
    // own requests of this step landed; behind the barrier everybody's, and everybody is done with the other two slots
    __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(0));
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (st + 1 < nst) {
      request(st + 1, next_page);
      next_page = bt[min(2 * (st + 2) + par, npg - 1)];
    }
    return &lds[0][0] + ((st & 1) * 2 + par) * (CH * 64) + lane;
  };
  // (pages before the block and pages reaching into it in loops of their own, so that neither variant carries the other)
  int st = 0;
  for (; 2 * st + 1 < first_masked; ++st) {
    const u32x4* L = open_step(st);
    if (has[0]) page_step(std::false_type{}, L, 2 * st + par);
  }
  for (; st < nst; ++st) {
    const u32x4* L = open_step(st);
    if (has[0] && 2 * st + par < npg) page_step(std::true_type{}, L, 2 * st + par);
  }
  // the odd pages' partials through LDS to the waves of the even pages
  __syncthreads();
  f32x4* po = (f32x4*)&lds[0][0] + qg * (2 * DT * 64) + lane;
  if (par == 1 && has[0]) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      ml[qg][i][lane] = make_float2(mrun[i], lacc[i][0]);
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) po[(i * DT + dt) * 64] = o[i][dt];
    }
  }
  __syncthreads();
  if (par == 1 || !has[0]) return;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int qrow = (qt0 + 2 * qg + i) * 16 + qc;
    const float2 t = ml[qg][i][lane];
    const float mm = fmaxf(mrun[i], t.x), ms = mm == -INFINITY ? 0.f : mm;
    const float f0 = __builtin_amdgcn_exp2f(mrun[i] - ms), f1 = __builtin_amdgcn_exp2f(t.x - ms);
    const float inv = 1.0f / (lacc[i][0] * f0 + t.y * f1), a0 = f0 * inv, a1 = f1 * inv;
    if (qrow >= nq) continue;
    const int row = seq_row0[b] + qrow / rep, col0 = (kvh * rep + qrow % rep) * D + 4 * g;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
      const f32x4 x = po[(i * DT + dt) * 64];
      *(uint2*)(out + act_offset(row, col0 + dt * 16, out_ktiles)) =
          make_uint2(pack2(o[i][dt][0] * a0 + x[0] * a1, o[i][dt][1] * a0 + x[1] * a1), pack2(o[i][dt][2] * a0 + x[2] * a1, o[i][dt][3] * a0 + x[3] * a1));
    }
  }
}

// ---------------------------------------------------------------------------------------------
// The same attention for few query rows over short contexts (drafted and catch-up rows, verify blocks of a batch): latency,
// not bytes, bounds these calls.  A workgroup takes one q-tile of one KV head and a run of `per` pages; its eight waves take
// every eighth page each, straight from HBM / L2 into registers (no LDS staging, no barrier per page: 256 KiB in flight per
// compute unit), and meet once in LDS at the end.  The q-tiles of a KV head read the same pages from one L2 (blockIdx.x is
// the KV head).  Up to a few pages per wave the call is then one launch, where the kernel above needs KV splits and a merge.
// ---------------------------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(512) void attn_tile_kernel(const uint4* __restrict__ Q, const bf16_t* __restrict__ kv, const int* seq_m,
                                                        const int* seq_p0, const int* seq_row0, const int* qt_seq, const int* qt_local,
                                                        const int* block_table, int pos_add, int rep, int Hkv, int layer, int n_pages,
                                                        int pps, int nsplit, int per, float* part_o, float* part_ml,
                                                        bf16_t* __restrict__ out, int out_ktiles) {
  constexpr int DS = D / 32, DT = D / 16, KCH = 4 * DS;
  __shared__ f32x4 lo[8][DT][64];
  __shared__ float2 ml[8][64];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), g = lane >> 4, qc = lane & 15;
  const int kvh = blockIdx.x, gqt = blockIdx.y, sp = blockIdx.z;
  const int b = qt_seq[gqt], qt = qt_local[gqt], total_qt = gridDim.y;
  const int m = seq_m[b], p0 = seq_p0[b] + pos_add, row0 = seq_row0[b], nq = m * rep, kv_end = p0 + m;
  const int npages = (kv_end + EE_PAGE - 1) / EE_PAGE, pg0 = sp * per, pg1 = min(npages, pg0 + per);
  if (pg0 >= npages) return;                            // whole workgroup; the merge pass knows this sequence's split count
  const int* bt = block_table + b * pps;
  const int qrow = qt * 16 + qc, limit = qrow < nq ? p0 + qrow / rep : -1;
  u32x4 qf[DS];
#pragma unroll
  for (int s = 0; s < DS; ++s) qf[s] = ((const u32x4*)Q)[(((size_t)kvh * total_qt + gqt) * DS + s) * 64 + lane];
  const float sc2 = 1.4426950408889634f / sqrtf((float)D);         // scores in base-2 units, as above
  const u32x4 ones = {0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u};
  float mrun = -INFINITY;
  f32x4 o[DT], lacc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) o[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
  u32x4 kf[KCH], vf[2 * DT];
  auto page_ptr = [&](int pg) __attribute__((always_inline)) {
    return (const u32x4*)(kv + kv_slab(layer, bt[pg], kvh, n_pages, Hkv, D)) + lane;
  };
  int pg = pg0 + wave;
  const u32x4* src = page_ptr(min(pg, pg1 - 1));
  if (pg < pg1) {
#pragma unroll
    for (int c = 0; c < KCH; ++c) kf[c] = __builtin_nontemporal_load(src + c * 64);
#pragma unroll
    for (int c = 0; c < 2 * DT; ++c) vf[c] = __builtin_nontemporal_load(src + (KCH + c) * 64);
  }
  for (; pg < pg1; pg += 8) {
    const int base = pg * EE_PAGE + 16 * g;             // this lane group holds positions base .. base+15
    // (the next page's fragments are requested as soon as this page's are consumed; past the end the last page again, unused)
    const u32x4* nsrc = page_ptr(min(pg + 8, pg1 - 1));
    f32x4 s4[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) s4[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < DS; ++s)
#pragma unroll
      for (int t = 0; t < 4; ++t) s4[t] = mfma16(kf[t * DS + s], qf[s], s4[t]);
    if (pg + 8 < pg1) {
#pragma unroll
      for (int c = 0; c < KCH; ++c) kf[c] = __builtin_nontemporal_load(nsrc + c * 64);
    }
    const bool masked = (pg + 1) * EE_PAGE > p0;        // reaches into the block or past the end (uniform)
    float tmax = -INFINITY;
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        if (base + 4 * t + v > limit) s4[t][v] = -INFINITY;
        tmax = fmaxf(tmax, s4[t][v]);
      }
    tmax = colmax4(tmax * sc2);
    const float mnew = fmaxf(mrun, tmax);
    const float msafe = mnew == -INFINITY ? 0.f : mnew;
    const float alpha = __builtin_amdgcn_exp2f(mrun - msafe), nm = -msafe;
    mrun = mnew;
    uint32_t pk[8];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      pk[2 * t] = pack2(__builtin_amdgcn_exp2f(fmaf(s4[t][0], sc2, nm)), __builtin_amdgcn_exp2f(fmaf(s4[t][1], sc2, nm)));
      pk[2 * t + 1] = pack2(__builtin_amdgcn_exp2f(fmaf(s4[t][2], sc2, nm)), __builtin_amdgcn_exp2f(fmaf(s4[t][3], sc2, nm)));
    }
    if (__builtin_amdgcn_ballot_w64(alpha != 1.0f) != 0) {
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) { o[dt][0] *= alpha; o[dt][1] *= alpha; o[dt][2] *= alpha; o[dt][3] *= alpha; }
      lacc[0] *= alpha; lacc[1] *= alpha; lacc[2] *= alpha; lacc[3] *= alpha;
    }
    const u32x4 P[2] = {u32x4{pk[0], pk[1], pk[2], pk[3]}, u32x4{pk[4], pk[5], pk[6], pk[7]}};
    if (masked) {      // dead positions (>= kv_end) may hold anything: zero their V
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int pa = base + 8 * ks + 2 * j;
          const uint32_t keep = pa + 1 < kv_end ? 0xffffffffu : (pa < kv_end ? 0xffffu : 0u);
#pragma unroll
          for (int dt = 0; dt < DT; ++dt) vf[dt * 2 + ks][j] &= keep;
        }
    }
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      lacc = mfma16(ones, P[ks], lacc);
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) o[dt] = mfma16(vf[dt * 2 + ks], P[ks], o[dt]);
    }
    if (pg + 8 < pg1) {
#pragma unroll
      for (int c = 0; c < 2 * DT; ++c) vf[c] = __builtin_nontemporal_load(nsrc + (KCH + c) * 64);
    }
  }
  ml[wave][lane] = make_float2(mrun, lacc[0]);
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) lo[wave][dt][lane] = o[dt];
  __syncthreads();
  if (wave >= DT) return;                               // wave w finishes d-tile w, in a fixed order over the waves
  float mall = -INFINITY, f[8], l = 0.f;
#pragma unroll
  for (int w = 0; w < 8; ++w) mall = fmaxf(mall, ml[w][lane].x);
  const float msafe = mall == -INFINITY ? 0.f : mall;
  f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int w = 0; w < 8; ++w) {
    const float2 t = ml[w][lane];
    f[w] = __builtin_amdgcn_exp2f(t.x - msafe);
    l += f[w] * t.y;
    const f32x4 x = lo[w][wave][lane];
    acc[0] += f[w] * x[0]; acc[1] += f[w] * x[1]; acc[2] += f[w] * x[2]; acc[3] += f[w] * x[3];
  }
  if (nsplit == 1) {
    if (qrow < nq) {
      const float inv = 1.0f / l;
      const int row = row0 + qrow / rep, col = (kvh * rep + qrow % rep) * D + wave * 16 + 4 * g;
      *(uint2*)(out + act_offset(row, col, out_ktiles)) = make_uint2(pack2(acc[0] * inv, acc[1] * inv), pack2(acc[2] * inv, acc[3] * inv));
    }
  } else {
    const size_t slot = ((size_t)gqt * Hkv + kvh) * nsplit + sp;
    if (wave == 0 && g == 0) *(float2*)(part_ml + slot * 32 + qc * 2) = make_float2(mall, l);
    ((f32x4*)part_o)[(slot * DT + wave) * 64 + lane] = acc;
  }
}

// merge the KV splits of one (q-tile, KV head) and emit the bf16 attention output in fragment layout
// (O-projection operand).  Workgroup = (q-tile, KV head, pair of d-tiles); its four waves share out the
// splits (wave w takes w, w+4, ...), each folding its share with all loads of a batch of eight splits in
// flight at once, and the four wave results meet in LDS.  Every lane owns the accumulator elements the
// split kernel's lanes did, so partials are read as coalesced float4.
template <int D>
__global__ __launch_bounds__(256) void attn_merge_kernel(const float* __restrict__ part_o, const float* __restrict__ part_ml,
                                                         const int* qt_seq, const int* qt_local, const int* seq_m,
                                                         const int* seq_p0, const int* seq_row0, int pos_add, int rep, int Hkv,
                                                         int slot_stride, int per, bf16_t* __restrict__ out, int out_ktiles) {
  constexpr int DT = D / 16, DW = 2;         // d-tiles per workgroup; gridDim.z = DT / DW
  __shared__ float sm[4][64], sd[4][64];
  __shared__ f32x4 sacc[4][DW][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, g = lane >> 4, qc = lane & 15;
  const int gqt = blockIdx.x, kvh = blockIdx.y, dq = blockIdx.z;
  const int b = qt_seq[gqt], qt = qt_local[gqt];
  const int nq = seq_m[b] * rep, qrow = qt * 16 + qc;
  const int npages = (seq_p0[b] + pos_add + seq_m[b] + EE_PAGE - 1) / EE_PAGE;
  const int nsplit = (npages + per - 1) / per;          // this sequence's split count
  const size_t slot0 = ((size_t)gqt * Hkv + kvh) * slot_stride;
  const float2* ml = (const float2*)(part_ml + slot0 * 32) + qc;
  const f32x4* pi = (const f32x4*)part_o + slot0 * (DT * 64) + (size_t)dq * DW * 64 + lane;
  float mw = -INFINITY, den = 0.f;
  f32x4 acc[DW];
#pragma unroll
  for (int j = 0; j < DW; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int s0 = wave; s0 < nsplit; s0 += 32) {
    float2 t[8];
    f32x4 ov[8][DW];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int sl = min(s0 + 4 * i, nsplit - 1);
      t[i] = ml[sl * 16];
#pragma unroll
      for (int j = 0; j < DW; ++j) ov[i][j] = __builtin_nontemporal_load(pi + ((size_t)sl * DT + j) * 64);
    }
    float bm = mw;
#pragma unroll
    for (int i = 0; i < 8; ++i) bm = fmaxf(bm, s0 + 4 * i < nsplit ? t[i].x : -INFINITY);
    const float safe = bm == -INFINITY ? 0.f : bm;
    const float sc = __builtin_amdgcn_exp2f(mw - safe);
    den *= sc;
#pragma unroll
    for (int j = 0; j < DW; ++j) { acc[j][0] *= sc; acc[j][1] *= sc; acc[j][2] *= sc; acc[j][3] *= sc; }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float w = s0 + 4 * i < nsplit ? __builtin_amdgcn_exp2f(t[i].x - safe) : 0.f;
      den += w * t[i].y;
#pragma unroll
      for (int j = 0; j < DW; ++j) { acc[j][0] += w * ov[i][j][0]; acc[j][1] += w * ov[i][j][1]; acc[j][2] += w * ov[i][j][2]; acc[j][3] += w * ov[i][j][3]; }
    }
    mw = bm;
  }
  sm[wave][lane] = mw; sd[wave][lane] = den;
#pragma unroll
  for (int j = 0; j < DW; ++j) sacc[wave][j][lane] = acc[j];
  __syncthreads();
  if (wave != 0) return;
  float mall = -INFINITY;
#pragma unroll
  for (int w = 0; w < 4; ++w) mall = fmaxf(mall, sm[w][lane]);
  const float msafe = mall == -INFINITY ? 0.f : mall;
  den = 0.f;
#pragma unroll
  for (int j = 0; j < DW; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int w = 0; w < 4; ++w) {        // fixed order: the result does not depend on timing
    const float f = __builtin_amdgcn_exp2f(sm[w][lane] - msafe);
    den += f * sd[w][lane];
#pragma unroll
    for (int j = 0; j < DW; ++j) {
      const f32x4 a = sacc[w][j][lane];
      acc[j][0] += f * a[0]; acc[j][1] += f * a[1]; acc[j][2] += f * a[2]; acc[j][3] += f * a[3];
    }
  }
  if (qrow < nq) {
    const float inv = 1.0f / den;
    const int row = seq_row0[b] + qrow / rep, col0 = (kvh * rep + qrow % rep) * D + dq * DW * 16 + 4 * g;
#pragma unroll
    for (int j = 0; j < DW; ++j)
      *(uint2*)(out + act_offset(row, col0 + j * 16, out_ktiles)) =
          make_uint2(pack2(acc[j][0] * inv, acc[j][1] * inv), pack2(acc[j][2] * inv, acc[j][3] * inv));
  }
}

// Pages per KV split of attn_kernel.  Every split of every sequence takes the same number of pages, so that a ragged
// batch is cut into workgroups of equal length; the count is the smallest one that keeps the launch within one workgroup
// per compute unit (the LDS ring admits one resident workgroup, so a second round would start cold).  kv_end[b] = 0: sequence
// not taking part.
static int ring_pages_per_split(const int* kv_end, const int* seq_m, int B, int rep, int Hkv, int max_pages, int max_splits) {
  int per = max(2, ceil_div(max_pages, max(1, min(max_splits, EE_MAX_SPLITS))));
  if (g_attn_pages_override > 0) return min(max(per, g_attn_pages_override), max_pages);   // (never more splits than the scratch holds)
  for (; per < max_pages; ++per) {
    long wgs = 0;
    for (int b = 0; b < B; ++b)
      if (kv_end[b] > 0)
        wgs += (long)ceil_div(ceil_div(kv_end[b], EE_PAGE), per) * Hkv * ceil_div(ceil_div(seq_m[b] * rep, 16), EE_ATTN_COMPUTE);
    if (wgs <= 256) break;
  }
  return min(per, max_pages);
}

// Kernel and split length of a call.  Long blocks that fill the chip unsplit take attn_block_kernel: in a context build
// always (it stops at a block's last page; one page is quicker in the ring, 8.0 us against 9.8), behind a longer context
// if it needs fewer rounds of workgroups -- it takes eight q-tiles where the ring takes six, for a quarter more a page (8B
// heads, 32 sequences behind 1000 positions: 7 / 9 / 13 q-tiles ring 56 / 57 / 83 us in 2 / 2 / 3 rounds, block 44 / 70 / 71 in
// 1 / 2 / 2; 8 behind 4000: 16 / 25 q-tiles ring 82 / 154, block 103 / 101).  Else the cheaper of the ring kernel and the tile
// kernel by what they measured (8B head shapes, head_dim 128, microseconds; a merge launch adds 5.8):
//   ring: 3 + 1.5 per page of a split                       (one sequence, 9 rows, 2 pages a split: 11.1 with the merge)
//   tile: 3.9 + 0.52 per page a workgroup reads -- one compute unit takes in no more than about 60 GB/s; more workgroups than
//         compute units take their sum over the chip and 30 % (2 pages 4.6, 8 pages 7.7, 16 pages 12.3; 384 workgroups of 16
//         pages on average 26.9)
// and neither quicker than the bytes at 6.5 TB/s.  Eight requests of ~1000 tokens, one row each: ring 16.9, tile 12.7; one
// request, 500 tokens, 9 rows: 9.7 / 7.6; one request, 2048 tokens, 9 rows: 11.1 / 11.8.  The tile kernel never takes more
// splits than the ring kernel would, so the scratch of a call does not grow, and has to promise 5 %.  A pinned split length
// (test hook) keeps every call in the ring kernel, so that a sequence is cut alike alone and in a batch.
AttnPlan bf16_attention_plan(const int* kv_end, const int* seq_m, int B, int Hq, int Hkv, int max_splits) {
  const int rep = Hq / Hkv;
  int max_pages = 1, max_qt = 0;
  long pages = 0;
  for (int b = 0; b < B; ++b) {
    if (kv_end[b] <= 0) continue;
    const int n = ceil_div(kv_end[b], EE_PAGE);
    max_pages = max(max_pages, n); max_qt = max(max_qt, ceil_div(seq_m[b] * rep, 16));
    pages += n;
  }
  AttnPlan ring{ATTN_RING, ring_pages_per_split(kv_end, seq_m, B, rep, Hkv, max_pages, max_splits), 1};
  ring.nsplit = ceil_div(max_pages, ring.per);
  if (g_attn_form == ATTN_RING) return ring;
  if (g_attn_form > ATTN_RING) return AttnPlan{g_attn_form, max_pages, 1};      // (both serve any call unsplit)
  if (g_attn_pages_override > 0) return ring;
  if (ring.nsplit == 1 && max_qt > EE_ATTN_COMPUTE && max_pages > 1) {
    long rows = 0, cached = 0, wg_ring = 0, wg_block = 0;
    for (int b = 0; b < B; ++b) {
      if (kv_end[b] <= 0) continue;
      const int q = ceil_div(seq_m[b] * rep, 16);
      rows += seq_m[b]; cached += kv_end[b] - seq_m[b];
      wg_ring += (long)Hkv * ceil_div(q, EE_ATTN_COMPUTE); wg_block += (long)Hkv * ceil_div(q, 8);
    }
    if (rows >= cached || 4 * ((wg_ring + 255) / 256) >= 5 * ((wg_block + 255) / 256)) return AttnPlan{ATTN_BLOCK, max_pages, 1};
  }
  const float floor_us = pages * Hkv * (EE_PAGE * 128 * 4.0f) / 6.5e6f, merge_us = 5.8f;
  float least = max(3.0f + 1.5f * ring.per, floor_us) + (ring.nsplit > 1 ? merge_us : 0.f);
  AttnPlan best = ring;
  for (int per = 8;; per += 8) {
    per = min(per, max_pages);
    const int nsplit = ceil_div(max_pages, per);
    if (nsplit <= ring.nsplit) {
      long wgs = 0, reads = 0;                         // workgroups, pages they read
      for (int b = 0; b < B; ++b) {
        if (kv_end[b] <= 0) continue;
        const int n = ceil_div(kv_end[b], EE_PAGE), q = ceil_div(seq_m[b] * rep, 16) * Hkv;
        wgs += (long)ceil_div(n, per) * q; reads += (long)n * q;
      }
      const float whole = (3.9f * wgs + 0.52f * reads) / 256.0f;
      const float us = max(max(3.9f + 0.52f * per, wgs > 256 ? 1.3f * whole : 0.f), floor_us) + (nsplit > 1 ? merge_us : 0.f);
      if (us < 0.95f * least) { least = us; best = AttnPlan{ATTN_TILE, per, nsplit}; }
    }
    if (per >= max_pages) break;
  }
  return best;
}

template <int D>
static void launch_attn(hipStream_t st, const AttnPlan& plan, const bf16_t* Q, const bf16_t* kv, const CallMeta& meta, int pos_add, int B,
                        int max_qt, int rep, int total_qt, int Hkv, int layer, int n_pages, int pps, const AttnScratch& scr, bf16_t* out,
                        int out_ktiles) {
  if (plan.kind == ATTN_BLOCK) {
    hipLaunchKernelGGL((attn_block_kernel<D>), dim3(Hkv, ceil_div(max_qt, 8), B), dim3(512), 0, st, (const uint4*)Q, kv, meta.seq_m,
                       meta.seq_p0, meta.seq_qt0, meta.seq_row0, meta.block_table, pos_add, rep, total_qt, Hkv, layer, n_pages, pps, out,
                       out_ktiles);
    return;
  }
  if (plan.kind == ATTN_TILE)
    hipLaunchKernelGGL((attn_tile_kernel<D>), dim3(Hkv, total_qt, plan.nsplit), dim3(512), 0, st, (const uint4*)Q, kv, meta.seq_m,
                       meta.seq_p0, meta.seq_row0, meta.qt_seq, meta.qt_local, meta.block_table, pos_add, rep, Hkv, layer, n_pages, pps,
                       plan.nsplit, plan.per, scr.part_o, scr.part_ml, out, out_ktiles);
  else
    hipLaunchKernelGGL((attn_kernel<D, 1>), dim3(plan.nsplit, Hkv * ceil_div(max_qt, EE_ATTN_COMPUTE), B), dim3(64 * EE_ATTN_WAVES), 0, st,
                       (const uint4*)Q, kv, meta.seq_m, meta.seq_p0, meta.seq_qt0, meta.seq_row0, meta.block_table, pos_add, rep,
                       total_qt, Hkv, layer, n_pages, pps, plan.nsplit, plan.per, scr.part_o, scr.part_ml, out, out_ktiles);
  if (plan.nsplit > 1)
    hipLaunchKernelGGL((attn_merge_kernel<D>), dim3(total_qt, Hkv, D / 32), dim3(256), 0, st, scr.part_o, scr.part_ml, meta.qt_seq,
                       meta.qt_local, meta.seq_m, meta.seq_p0, meta.seq_row0, pos_add, rep, Hkv, plan.nsplit, plan.per, out, out_ktiles);
}

void bf16_attention(hipStream_t st, const AttnPlan& plan, const bf16_t* Q, const bf16_t* kv, const CallMeta& meta, int pos_add, int B,
                    int max_m, int total_qt, int Hq, int Hkv, int D, int layer, int n_pages, int pages_per_seq, const AttnScratch& scr,
                    bf16_t* out, int out_ktiles) {
  const int rep = Hq / Hkv, max_qt = ceil_div(max_m * rep, 16);
  if (D == 128) launch_attn<128>(st, plan, Q, kv, meta, pos_add, B, max_qt, rep, total_qt, Hkv, layer, n_pages, pages_per_seq, scr, out, out_ktiles);
  else launch_attn<64>(st, plan, Q, kv, meta, pos_add, B, max_qt, rep, total_qt, Hkv, layer, n_pages, pages_per_seq, scr, out, out_ktiles);
}
