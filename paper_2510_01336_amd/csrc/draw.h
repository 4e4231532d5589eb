// Decisions of the inverse-CDF draw (kernels_sample.hip): which group of chunks and which token a target falls into.  Host and
// device, so that a host program can put them through the sums a wave forms.
// The cumulative weights of lanes and groups come from tree scans: two neighbouring prefixes are rounded along different paths,
// so a prefix may already exceed the target before its own first weight is added, and prefixes need not even rise.  A place is
// therefore admitted only if it carries weight itself: a token of weight zero -- in a residual draw the token just rejected and
// about half of the vocabulary -- is never drawn.
#pragma once
#include <hip/hip_runtime.h>

// a group of chunks of weight `group`, whose inclusive prefix ends at `incl`
__host__ __device__ inline bool draw_admits_group(float incl, float group, float target) { return group > 0.f && incl > target; }

// among four consecutive weights behind the prefix `base`: the first with weight whose cumulative weight exceeds the target; 4: none
__host__ __device__ inline int draw_among_four(float base, float4 x, float target) {
  const float s0 = x.x, s1 = s0 + x.y, s2 = s1 + x.z, s3 = s2 + x.w;
  if (x.x > 0.f && base + s0 > target) return 0;
  if (x.y > 0.f && base + s1 > target) return 1;
  if (x.z > 0.f && base + s2 > target) return 2;
  return x.w > 0.f && base + s3 > target ? 3 : 4;
}

// the last of four consecutive places that carries weight; -1: none
__host__ __device__ inline int draw_last_of_four(float4 x) { return x.w > 0.f ? 3 : (x.z > 0.f ? 2 : (x.y > 0.f ? 1 : (x.x > 0.f ? 0 : -1))); }
