// Row factors rsqrt(mean(x^2) + eps) of the deferred RMSNorm from the producer's partial sums of squares [partial][row], as a launch of its
// own (calls and parts of more than 192 rows).
#pragma once
#include "common.h"

// The order in which a row's partials are added: 64 chains (chain t takes partials t, t + 64, t + 128, ...) of four sums each, which take whole
// turns of four; what is left of the last turn goes to the first sum.  Then a tree over the four sums and over neighbouring chains.  Up to 16
// partials that is also the order of norm_factors (kernels_bf16.hip), which has 16 chains; beyond, the two differ in the last bits.
// The turn that starts at partial i, of n: x[j] is partial i + 64 * j (any number where there is none).  Without a branch, so that the loads
// of several chains stay together: adding 0 leaves a sum of squares as it is.
__host__ __device__ inline void norm_chain_add(float (&s)[4], const float (&x)[4], int i, int n) {
  const bool whole = i + 192 < n;
  const float x0 = i < n ? x[0] : 0.f, x1 = i + 64 < n ? x[1] : 0.f, x2 = i + 128 < n ? x[2] : 0.f;
  s[0] = (s[0] + x0) + (whole ? 0.f : x1) + (whole ? 0.f : x2);
  s[1] += whole ? x1 : 0.f;
  s[2] += whole ? x2 : 0.f;
  s[3] += whole ? x[3] : 0.f;
}
__host__ __device__ inline float norm_chain_sum(const float (&s)[4]) { return (s[0] + s[1]) + (s[2] + s[3]); }
// sum of N (a power of two) neighbouring chains or groups of them, left in t[0]
template <int N>
__host__ __device__ inline float norm_tree(float (&t)[N]) {
#pragma unroll
  for (int n = N / 2; n >= 1; n >>= 1)
#pragma unroll
    for (int w = 0; w < n; ++w) t[w] = t[2 * w] + t[2 * w + 1];
  return t[0];
}

// A workgroup takes 32 rows, so that a load reads two runs of 128 bytes, and its sixteen waves four chains each, two a lane: the eight loads of
// a turn are requested ahead of the first add (repeats of the last partial behind it).  What bounds it is the launch and one trip to memory for
// every 256 partials.  One launch behind another, us, with a wave per row and lanes along the partials, which reads sixteen bytes of every
// line, and now (the same bits): 512 rows, 64 partials 2.31 / 2.32, 128 2.68 / 2.32, 192 3.04 / 2.31, 320 3.32 / 2.71; 1096 rows, 256 partials
// 4.24 / 2.33; 2048 rows 5.43 / 2.34; 4096 rows 8.6 / 2.58, 320 partials 10.5 / 3.1.  (With the loads of a turn one behind another wherever the
// turn is not whole, 192 partials took 0.8 us more than with a wave per row.)
#define EE_NORM_ROWS 32      // rows of a workgroup
__global__ __launch_bounds__(1024) void norm_factor_kernel(const float* __restrict__ ssq, int n_part, int stride, float inv_d, float eps,
                                                           float* __restrict__ inv_rms, int M) {
  __shared__ float sum[16][EE_NORM_ROWS];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r = lane & 31, row = blockIdx.x * EE_NORM_ROWS + r;
  const int t0 = 4 * wave + 2 * (lane >> 5);      // the lane's chains: t0 and its neighbour
  const float* p = ssq + min(row, M - 1);
  float s[2][4];
#pragma unroll
  for (int c = 0; c < 2; ++c) s[c][0] = s[c][1] = s[c][2] = s[c][3] = 0.f;
  for (int i0 = 0; i0 < n_part; i0 += 256) {
    float x[2][4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int c = 0; c < 2; ++c) x[c][j] = p[(size_t)min(i0 + t0 + c + 64 * j, n_part - 1) * stride];
#pragma unroll
    for (int c = 0; c < 2; ++c) norm_chain_add(s[c], x[c], i0 + t0 + c, n_part);
  }
  float y = norm_chain_sum(s[0]) + norm_chain_sum(s[1]);
  y += __shfl_xor(y, 32, 64);
  if (lane < 32) sum[wave][r] = y;
  __syncthreads();
  if (threadIdx.x >= EE_NORM_ROWS || row >= M) return;
  float t[16];
#pragma unroll
  for (int w = 0; w < 16; ++w) t[w] = sum[w][r];
  inv_rms[row] = 1.0f / sqrtf(norm_tree(t) * inv_d + eps);
}
