// Launch shapes of the few-row GEMM (gemm_skinny_kernel): which strips of weight tiles go to which wave.  Pure functions of the sizes,
// so that a host program can put every size through them.
#pragma once
#include "common.h"
#include <algorithm>

struct StripShape { int ns, nw, ksplit, U; };   // strips per wave, waves per workgroup, waves that share out K, k-tiles per register set

// strips (weight tiles) on the busiest compute unit when workgroups take per_wg each
inline int strip_load(int ntiles, int per_wg) { return ceil_div(ceil_div(ntiles, per_wg), 256) * per_wg; }
// 128 MB and more of weights
inline bool strips_large(int ntiles, int ktiles) { return (size_t)ntiles * ktiles * 1024 >= ((size_t)128 << 20); }

// K shares of a strip.  Below 128 MB they are a matter of the matrix alone: a row's sums then run over K in one order and are the same
// bits however many rows are beside it (up to EE_STRIP_ROWS).  A large wide matrix is summed over the whole K by one wave up to 16 rows,
// where a wave has one strip, and in eight shares beyond, where it has seven.
//   Eight for some 256 strips with a long K, 8B down at 9 / 24 rows 20.9 / 27.1 us (four 22.0 / 26.5), else four, never of fewer than four
//   k-tiles.
inline int strip_parts(int ntiles, int ktiles) {
  if (ntiles >= 768) return 1;
  if (ntiles > 512) return 8;
  int parts = ntiles >= 200 && ntiles < 320 && ktiles >= 256 ? 8 : 4;
  while (ntiles < 320 && parts > 1 && ktiles / parts < 4) parts >>= 1;
  return parts;
}

// Launch shape for M <= 32 rows, from sweeps over the matrices of the 8B and 70B widths with cold weights (us; {strips, waves,
// K parts, U}).  What bounds them is the memory path of a compute unit, which takes in weights and rows together at 35-50 GB/s,
// so the shape has to give every compute unit the same share of the strips and, with several strips a wave, read the rows less
// often.  `load`: strips on the busiest compute unit.
//   wide (>= 768 strips): a strip per wave, as many waves a workgroup as deal the strips most evenly: gate/up at 9 rows 8B 40.0
//     with four waves on 224 units, 38.9 with seven on 256; 70B 148 / 141.  At 17..32 rows of a large matrix seven strips a wave and
//     K over eight waves where that deals them evenly too (the rows are then read once for seven strips): 8B 40.3, 70B 144 (row-tiled
//     kernel 44.2, 147); else one strip a wave: head of 32000 tokens 47.9 (50.3).
//   narrow: K over four or eight waves.  Two or four strips a wave where that makes load * (1 + row tiles / strips) smaller: 70B
//     QKV (640 strips) at 9 / 24 rows 32.8 / 37.9 with four, 35.1 / 41.6 with one; 70B down 70.2 / 74.4 with two, 77.4 / 92.6; 8B
//     QKV (384) 13.3 / 15.5 with two, 13.8 / 16.6.  At one row tile, strips that fill the chip evenly and a K below 512 k-tiles stay
//     at one a wave (70B O 25.9 / 27.0).
inline StripShape strip_shape(int ntiles, int ktiles, int M) {
  const int mt = M > 16 ? 2 : 1, parts = strip_parts(ntiles, ktiles);
  if (ntiles >= 768) {
    if (mt == 2 && strips_large(ntiles, ktiles) && 256 * strip_load(ntiles, 7) <= ntiles * 23 / 20) return StripShape{7, 8, 8, 1};
    int nw = 8;
    for (int w = 7; w >= 4; --w)
      if (strip_load(ntiles, w) < strip_load(ntiles, nw)) nw = w;
    return StripShape{1, nw, 1, mt == 2 ? 4 : 8};
  }
  int ns = 1;
  if (ntiles >= 320 && (mt == 2 || ntiles % 256 != 0 || ktiles >= 512))
    for (int n = 2; n <= 4; n *= 2)
      if (strip_load(ntiles, n) * (n + mt) * ns < strip_load(ntiles, ns) * (ns + mt) * n) ns = n;
  if (ns == 4) return StripShape{4, 8, parts, mt == 2 ? 2 : 4};
  if (ns == 2) return StripShape{2, 4, parts, 4};
  return StripShape{1, std::max(4, parts), parts, mt == 2 ? 4 : 8};
}
