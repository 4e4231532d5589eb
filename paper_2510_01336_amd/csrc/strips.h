// Launch shapes of the few-row GEMM (gemm_skinny_kernel): which strips of weight tiles go to which wave; order of the blocks of the
// blocked one.  Pure functions of the sizes, so that a host program can put every size through them.
#pragma once
#include "common.h"
#include <algorithm>

#define EE_STRIP_ROWS 32   // most rows of a call of the few-row GEMM
#define EE_ROWS_TN 4       // weight tiles a wave of the row-tiled GEMM takes (a workgroup: twice as many)
struct StripShape { int ns, nw, ksplit; };   // strips per wave, waves per workgroup, waves that share out K

// strips (weight tiles) on the busiest compute unit when workgroups take per_wg each
inline int strip_load(int ntiles, int per_wg) { return ceil_div(ceil_div(ntiles, per_wg), 256) * per_wg; }
// 128 MB and more of weights
inline bool strips_large(int ntiles, int ktiles) { return (size_t)ntiles * ktiles * 1024 >= ((size_t)128 << 20); }

// number of K shares the row-tiled GEMM runs with: enough workgroups for the chip, at least 16 k-tiles each
inline int rows_ksplit(int ntiles, int ktiles) {
  const int groups = ceil_div(ntiles, 2 * EE_ROWS_TN);
  int ks = groups >= 192 ? 1 : std::min(8, ceil_div(224, groups));
  while (ks > 1 && ktiles / ks < 16) --ks;
  return ks;
}
// A call of 17..32 rows of a large matrix goes to the few-row GEMM or to the row-tiled one, whichever measured faster (one launch behind
// another, cold weights, us at 17 / 24 / 32 rows, strips against row-tiled with its reduction; n x k: weight tiles x k-tiles):
//   wide, seven strips a wave (the rows are read once for seven strips, which is worth a third more than an even share on the busiest
//     compute unit): gate/up 8B 39.9 / 39.9 / 40.0 (44.3), 70B 145 / 146 / 147 (149), 1376 x 128 32.4 / 32.6 / 32.9 (49.3), 2752 x 256
//     121 / 122 / 125 (131); head of 128256 tokens 8B 175 / 179 / 183 (185 / 187 / 189), 70B 328 / 333 / 340 (333 / 336 / 340).  The row-tiled
//     kernel suffers where K is a multiple of 2048, so that all its strips start at one place of the memory channels; where it is
//     not, a head of many rounds is quicker there: 8016 x 96 143 / 146 / 149 (133 / 134 / 136), 9496 x 80 149 / 152 / 156 (144 / 146 / 148)
//   wide, one strip a wave, where the row-tiled kernel would need K shares (960 x 160 32.7 / 32.9 / 35.0, 34.0) or K is short and
//     either a multiple of 2048 (2000 x 128 46.0 / 48.0 / 51.4, 50.6; 3000 x 64 37.5 / 38.1 / 39.8, 50.4) or the row-tiled kernel's last
//     round half empty (2368 x 112 56.4 / 57.4 / 60.6, 61.1); not 2000 x 96 36.4 / 37.7 / 40.0 (35.7), 2000 x 160 57.4 / 60.4 / 65.0 (56.0),
//     2000 x 256 89 / 96 / 103 (87)
//   narrow, where pairs of strips are an even deal: 70B O 28.4 / 28.9 / 29.3 (32.0); of a long K, where the rows outgrow the weights, up
//     to 20 rows: 70B down 73.0 / 76.4 / 81.0 (75.1), 512 x 688 60.7 / 62.4 / 65.5 (61.5).  Never uneven ones: 70B QKV 37.9 / 38.7 / 39.9
//     (37.2), 13B down 31.9 / 34.0 / 36.4 (26.9)
inline bool strips_by_seven(int ntiles, int ktiles) {
  const int load = strip_load(ntiles, 7);
  return strips_large(ntiles, ktiles) && ntiles >= 768 && 3 * 256 * load <= 4 * ntiles && (ktiles % 64 == 0 || load <= 28);
}
// whether the few-row GEMM serves a call of M rows: up to 16 of any matrix, up to 32 of those below 128 MB, else as above
inline bool strips_serve(int ntiles, int ktiles, int M) {
  if (M <= 16 || !strips_large(ntiles, ktiles)) return M <= EE_STRIP_ROWS;
  if (M > EE_STRIP_ROWS) return false;
  if (ntiles < 768) return 256 * strip_load(ntiles, 2) <= ntiles * 23 / 20 && (ktiles < 512 || M <= 20);
  if (strips_by_seven(ntiles, ktiles) || rows_ksplit(ntiles, ktiles) > 1) return true;
  const int groups = ceil_div(ntiles, 2 * EE_ROWS_TN);
  const bool rows_even = ceil_div(groups, 256) * 256 <= groups * 23 / 20;
  return ktiles <= 128 && (ktiles % 64 == 0 || !rows_even);
}

// K shares of a strip.  Below 128 MB they are a matter of the matrix alone: a row's sums then run over K in one order and are the same
// bits however many rows are beside it (up to EE_STRIP_ROWS).  A large wide matrix is summed over the whole K by one wave up to 16 rows,
// where a wave has one strip, and in eight shares beyond, where it has seven.
//   Four, never of fewer than four k-tiles; eight on around 256 strips of 416 to 511 k-tiles, where single rows, most of a decoding
//   step, gain more than 17..32 lose: us at 1 / 9 / 24 rows, eight and four, 256 x 448 (8B down) 19.8 / 21.1 / 27.2, 20.5 / 21.1 / 26.5;
//   256 x 432 19.3 / 20.8 / 26.5, 19.6 / 20.9 / 25.5; but 256 x 344 17.9 / 18.9 / 22.2, 16.7 / 17.7 / 22.0; 256 x 400 18.8 / 20.2 / 24.7, 18.3 / 19.5 / 24.0;
//   256 x 512 25.6 / 27.2 / 30.6, 25.4 / 27.2 / 31.1; 256 x 608 26.4 / 28.5 / 34.9, 25.6 / 27.3 / 34.4; 224 x 592 23.5 / 26.7 / 33.9, 22.6 / 25.9 / 32.9
inline int strip_parts(int ntiles, int ktiles) {
  if (ntiles >= 768) return 1;
  if (ntiles > 512) return 8;
  int parts = ntiles >= 200 && ntiles < 320 && ktiles >= 416 && ktiles < 512 ? 8 : 4;
  while (ntiles < 320 && parts > 1 && ktiles / parts < 4) parts >>= 1;
  return parts;
}

// Launch shape for M <= 32 rows, from sweeps over the matrices of the 8B and 70B widths with cold weights (us).  What bounds them is
// the memory path of a compute unit, which takes in weights and rows together at 35-50 GB/s, so the shape has to give every
// compute unit the same share of the strips and, with several strips a wave, read the rows less often.  `load`: strips on the busiest compute unit.
//   wide (>= 768 strips): a strip per wave, as many waves a workgroup as deal the strips most evenly: gate/up at 9 rows 8B 40.0
//     with four waves on 224 units, 38.9 with seven on 256; 70B 148 / 141.  Of equal deals four waves, whose workgroups start and end
//     sooner, where K is short (8016 x 64 at 9 rows 83.7, eight waves 92.0; 9496 x 80 120, 125; 5000 x 96 75.3, five 85.0), eight where
//     it is long (8016 x 128 at 9 / 16 rows 163.7 / 166.1, four 164.7 / 167.9; 8016 x 256 309 / 311, four 321 / 329).  At 17..32 rows of a
//     large matrix seven strips a wave and K over eight waves, see above.
//   narrow: K over four or eight waves.  Two or four strips a wave where that makes load * (1 + row tiles / strips) smaller: 70B
//     QKV (640 strips) at 9 / 24 rows 32.8 / 37.9 with four, 35.1 / 41.6 with one; 70B down 70.2 / 74.4 with two, 77.4 / 92.6; 8B
//     QKV (384) 13.3 / 15.5 with two, 13.8 / 16.6.  At one row tile, strips that fill the chip evenly and a K below 512 k-tiles stay
//     at one a wave (70B O 25.9 / 27.0).
inline StripShape strip_shape(int ntiles, int ktiles, int M) {
  const int mt = M > 16 ? 2 : 1, parts = strip_parts(ntiles, ktiles);
  if (ntiles >= 768) {
    if (mt == 2 && strips_by_seven(ntiles, ktiles)) return StripShape{7, 8, 8};
    int nw = ktiles >= 128 && strip_load(ntiles, 8) <= strip_load(ntiles, 4) ? 8 : 4;
    for (int w = 5; w <= 8; ++w)
      if (strip_load(ntiles, w) < strip_load(ntiles, nw)) nw = w;
    return StripShape{1, nw, 1};
  }
  int ns = 1;
  if (ntiles >= 320 && (mt == 2 || ntiles % 256 != 0 || ktiles >= 512))
    for (int n = 2; n <= 4; n *= 2)
      if (strip_load(ntiles, n) * (n + mt) * ns < strip_load(ntiles, ns) * (ns + mt) * n) ns = n;
  if (ns == 4) return StripShape{4, 8, parts};
  if (ns == 2) return StripShape{2, 4, parts};
  return StripShape{1, std::max(4, parts), parts};
}

// Strips of a workgroup of a QKV projection whose last one is half a strip, 0: whole strips only.  One and a half or two and a half, where
// those are the even deal, by the waves that share out K and the norm's partial sums anyway, so that the sums stay the same bits.  Up to 16
// rows (8B, 384 strips, at 1 / 9 / 16 rows 11.6 / 12.0 / 12.4 us, two whole strips 12.7 / 12.6 / 12.8, but at 32 rows 15.6, 15.1; 70B, 640 strips,
// 30.0 / 30.5 / 31.0, four whole ones 30.6 / 31.6 / 32.3; 288 x 128 at 9 rows 10.6, 11.9; 560 x 64 9.7, 12.8; 352 x 160 13.3, 13.6).
inline int strips_half(int ntiles, int ktiles, int M) {
  const StripShape s = strip_shape(ntiles, ktiles, M);
  if (M > 16 || ktiles < 64 || s.nw != s.ksplit) return 0;
  if (ntiles > 256 && ntiles <= 384 && s.ksplit == 4) return 2;
  if (ntiles > 512 && ntiles <= 640 && s.ksplit == 8) return 3;
  return 0;
}

// Workgroups of such a launch, and the i-th of the ns strips of workgroup id: ids 8 apart, which run on one XCD, share 2 * ns - 1 strips and
// halve the last one (half_of).
inline int half_grid(int ntiles, int ns) { return 16 * ceil_div(ceil_div(ntiles, 2 * ns - 1), 8); }
__host__ __device__ inline int half_of(int id) { return (id >> 3) & 1; }
__host__ __device__ inline int half_strip_at(int id, int i, int ns) {
  return ((id >> 4) * 8 + (id & 7)) * (2 * ns - 1) + (i < ns - 1 ? half_of(id) * (ns - 1) + i : 2 * (ns - 1));
}

// Whether a row block in which `used` of rt row tiles hold rows runs as a full one (tiles behind the last repeat it): one of its four wave
// pairs has as many as in a full block either way, and the full form has no conditions (8B O, 9 of 12 row tiles used: 52 us, 59 with them)
__host__ __device__ constexpr bool block_full(int used, int rt) { return used > rt - 4; }

// Tiles of a stage that a wave of such a block requests: wave, wave + 8, ... of the weight tiles and, behind them, the row tiles in use
__host__ __device__ constexpr int block_requests(int wave, int wt, int used) { return (wt + used + 7 - wave) / 8; }

// Forms of the blocked kernel: weight and row tiles per workgroup, with the time of one k-tile when all compute units are busy, the
// share of it that is left when few are (%; the clock gives way under load), and the time of a block's start and end, in ns.
// Gate/up and the head, whose 1536 and more weight tiles always fill the chip, from sweeps over 8B shapes on random operands (gate/up at
// 4096 rows 705 us with 16 weight tiles, 798 with 12).  Their narrow blocks of rows lose: gate/up at 1096 rows 258 (16 x 16), 264 (16 x 8).
// Of 294 gate/up calls of six widths from 520 to 4096 rows the model names the quicker of the two forms or one within 3.5 % (0.05 % on average); with
// a light row block at a third of a step and its share of the rest it took up to 18 % longer (8B at 1040 rows 208 us in 12 weight tiles, 224 in 16;
// 70B at 576 rows 480 in 16, 530 in 12).
// Narrow matrices (QKV, O, down, adapters) from six forms x 49 calls of 520 to 4096 rows at ten widths (1B to 70B).  The form it names takes 0.1 %
// longer than the quickest one on average and 7 % at most, also on 80 further row counts.  (Fitted to the 8B and 70B widths alone: 26 % at most, 384 x 512
// tiles at 2600 rows 591 us in 16 x 16, 467 in 12 x 12; 320 x 432 at 1300 rows 184 in 12 x 12, 176 in 8 x 16.)  Small blocks cost more per product but let
// such a matrix fill the chip -- us with 16 x 16, 12 x 16 and 8 x 16 tiles alone, and with all six: 8B O at 768 / 1024 / 1200 / 1536 rows 57.8 / 59.4 / 62.3 / 61.8,
// 43.3 / 44.1 / 52.4 / 55.1; 8B down at 900 / 1152 rows 171 / 174, 117 / 152; 8B QKV at 600 / 960 / 1536 / 3072 rows 57 / 62 / 88 / 171, 43 / 55 / 73 / 145.
struct BlockForm { int wt, rt, step, idle, ends; };
inline constexpr BlockForm kWideForms[2] = {{16, 16, 740, 100, 6000}, {12, 16, 620, 100, 6000}};
inline constexpr BlockForm kNarrowForms[6] = {{16, 16, 727, 50, 27500}, {12, 16, 585, 63, 20600}, {8, 16, 413, 57, 14900},
                                          {12, 12, 448, 58, 16600}, {8, 12, 344, 59, 12300}, {8, 8, 261, 53, 8400}};
constexpr int kCusPerXcd = 32;
// Time of one launch by list scheduling of one XCD's blocks on its compute units (every XCD works on an equal run of
// them, see the kernel); a light row block costs three quarters of a step and its share of the rest.
inline int block_cost(const BlockForm& f, int ntiles, int ktiles, int M) {
  const int rblocks = ceil_div(M, 16 * f.rt), n = ceil_div(ceil_div(ntiles, f.wt) * rblocks, 8);
  const int used = ceil_div(M - (rblocks - 1) * 16 * f.rt, 16);
  const int step = f.step * (f.idle + (100 - f.idle) * n / (kCusPerXcd * ceil_div(n, kCusPerXcd))) / 100;
  const int full = ktiles * step + f.ends, part = block_full(used, f.rt) ? full : ktiles * (step * 3 / 4 + step * used / (4 * f.rt)) + f.ends;
  int free_at[kCusPerXcd] = {0}, end = 0;
  for (int i = 0; i < n; ++i) {
    int c = 0;
    for (int k = 1; k < kCusPerXcd; ++k)
      if (free_at[k] < free_at[c]) c = k;
    free_at[c] += i % rblocks == rblocks - 1 ? part : full;
    end = std::max(end, free_at[c]);
  }
  return end;
}
// Form of a blocked call: the cheapest by this model
inline const BlockForm& block_form(bool wide, int ntiles, int ktiles, int M) {
  const BlockForm* forms = wide ? kWideForms : kNarrowForms;
  const BlockForm* best = forms;
  int least = 0;
  for (int i = 0; i < (wide ? 2 : 6); ++i) {
    const int cost = block_cost(forms[i], ntiles, ktiles, M);
    if (!i || cost < least) { best = forms + i; least = cost; }
  }
  return *best;
}

// Whether a narrow matrix (QKV, O, down, adapters) runs blocked at M > 512 rows, else as parts of 512 rows in K shares and the rest.  K up to N: always
// (8B O / QKV at 520 rows 35.9 / 39.3 us, in parts 40.0 / 54; 70B 92.9 / 102.8, 97.9 / 106.7).  A longer K leaves few blocks with much to do: from 1025
// rows, or where blocks of 8 weight tiles fill the chip; and where blocks of 128 rows fit one round, from the row count at which they are the
// quicker ones.  They take the longer the more K exceeds N, and the less the emptier the last of them is (light: up to half), while K shares always
// fill the chip.  Down, us, blocks / parts at 690, 736, 768, 784, 880, 928 rows:
//   320 x 432 tiles  107 / 130, 123 / 136, 127 / 140
//   192 x 256         62 / 71, 71 / 75, 74 / 77, 59 / 76, 74 / 82, 60 / 87
//   256 x 448 (8B)   108 / 116, 124 / 122, 128 / 124, 104 / 126, 128 / 134, 111 / 140
//   128 x 256         60 / 61, 70 / 64, 73 / 66, 57 / 66, 73 / 72, 57 / 75
//   224 x 592        135 / 130, 156 / 134, 161 / 138, 134 / 140, 161 / 151, 133 / 157
//   320 x 864        221 / 209, 230 / 216, 237 / 224; 70B down at 520 / 700 / 900 rows 293 / 283, 344 / 322, 395 / 425
inline bool blocks_serve_narrow(int ntiles, int ktiles, int M) {
  const int groups = ceil_div(ntiles, 8);
  if (ktiles <= ntiles || M > 1024 || groups * ceil_div(M, 256) >= 256) return true;
  const bool light = (M - 1) % 128 < 64;
  const int first = 2 * ktiles <= 3 * ntiles ? 673 : ktiles < 2 * ntiles ? (light ? 673 : 769) : (light ? 769 : 897);
  return M >= first && groups * ceil_div(M, 128) <= 256;
}

// Order of the blocks of a blocked launch (gemm_block_kernel): an XCD (workgroup id mod 8) gets consecutive blocks of an order in which
// `run` row blocks share a weight group before the next group follows.  The 32 blocks that it works on side by side cover run row
// blocks and 32 / run weight groups, and run is chosen so that they are the least its L2 has to fetch: moving tiles is what takes the
// clock away (without its requests the gate/up kernel at 4096 rows runs at 1.91 GHz instead of 1.74).  All row blocks in one run / in runs
// as chosen, 8B, us: 4096 rows gate/up 683 / 672, QKV 197 / 184, O 141 / 135, down 357 / 345; 3072 rows 544 / 541, 145 / 136, 116 / 110, 317 / 304; 2048
// rows QKV 94 / 93, O 72 / 70, down 199 / 195 (gate/up stays in one run there).  With a light last row block all are in one run: else only some
// XCDs would get those (8B O at 1800 rows 62.4 / 65.0, 2400 rows 111 / 112).
struct BlockOrder { int cols, rblocks, run, share; };      // weight groups, row blocks, row blocks of a run, blocks of an XCD
inline BlockOrder block_order(int ntiles, int M, int wt, int rt) {
  const int rblocks = ceil_div(M, 16 * rt);
  BlockOrder o{ceil_div(ntiles, wt), rblocks, rblocks, ceil_div(ceil_div(ntiles, wt) * rblocks, 8)};
  if (!block_full(ceil_div(M - (rblocks - 1) * 16 * rt, 16), rt)) return o;
  for (int runs = 1, least = 0; runs <= rblocks; ++runs) {
    const int g = ceil_div(rblocks, runs), tiles = g * rt + ceil_div(32 * wt, g);
    if (runs == 1 || tiles < least) { least = tiles; o.run = g; }
  }
  return o;
}
struct BlockPlace { int col, row; };      // weight group (-1: no block), row block
__host__ __device__ inline BlockPlace block_place(const BlockOrder& o, int id) {
  const int b = (id & 7) * o.share + (id >> 3);
  if ((id >> 3) >= o.share || b >= o.cols * o.rblocks) return BlockPlace{-1, 0};
  const int at = b / (o.cols * o.run), left = b - at * o.cols * o.run, wide = o.rblocks - at * o.run < o.run ? o.rblocks - at * o.run : o.run;
  return BlockPlace{left / wide, at * o.run + left % wide};
}
