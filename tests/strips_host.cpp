// Host program behind test_strips_host.py: the launch shapes of the few-row GEMM, the order and the requests of the blocked one (csrc/strips.h).
//   strips_host                          every matrix of up to 4200 strips: prints the sizes whose shape or order breaks a rule
//   strips_host gateup|other NTILES KTILES M   prints "weight-tiles row-tiles" of a workgroup of that blocked call
//   strips_host narrow NTILES KTILES M   prints "blocks" or "parts": form of a narrow matrix at more than 512 rows
//   strips_host NTILES KTILES M          prints "strips-per-wave waves K-parts" of that call, or "rows": not a call of this kernel
#include "../paper_2510_01336_amd/csrc/strips.h"
#include <cstdio>
#include <cstdlib>

int main(int argc, char** argv) {
  if (argc == 4) {
    const StripShape s = strip_shape(atoi(argv[1]), atoi(argv[2]), atoi(argv[3]));
    if (!strips_serve(atoi(argv[1]), atoi(argv[2]), atoi(argv[3]))) printf("rows\n");
    else printf("%d %d %d\n", s.ns, s.nw, s.ksplit);
    return 0;
  }
  if (argc == 5 && argv[1][0] != 'n') {
    const BlockForm& f = block_form(argv[1][0] == 'g', atoi(argv[2]), atoi(argv[3]), atoi(argv[4]));
    printf("%d %d\n", f.wt, f.rt);
    return 0;
  }
  if (argc == 5) {
    printf("%s\n", blocks_serve_narrow(atoi(argv[2]), atoi(argv[3]), atoi(argv[4])) ? "blocks" : "parts");
    return 0;
  }
  int bad = 0;
  auto wrong = [&](int nt, int kt, int M, const char* what) { if (++bad <= 20) printf("%d strips, %d k-tiles, %d rows: %s\n", nt, kt, M, what); };
  for (int nt = 1; nt <= 4200; ++nt)
    for (int kt : {1, 2, 3, 5, 8, 9, 15, 16, 17, 31, 32, 64, 96, 112, 128, 255, 256, 344, 448, 512, 896})
      for (int M : {1, 9, 16, 17, 24, 32}) {
        if (strips_serve(nt, kt, 33) || !strips_serve(nt, kt, 16) || (!strips_large(nt, kt) && !strips_serve(nt, kt, 32))) wrong(nt, kt, M, "wrong kernel");
        if (!strips_serve(nt, kt, M)) continue;
        const StripShape s = strip_shape(nt, kt, M), one = strip_shape(nt, kt, 1);
        if (s.nw < 1 || s.nw > EE_MAX_WAVES || s.ksplit < 1 || s.nw % s.ksplit) wrong(nt, kt, M, "waves do not share out the strips");
        if (s.ns != 1 && s.ns != 2 && s.ns != 4 && !(s.ns == 7 && M > 16)) wrong(nt, kt, M, "no kernel for so many strips a wave");
        // the K shares, and the shares of the norm's partial sums (one a wave), set the order of a row's sums
        if (!strips_large(nt, kt) && (s.ksplit != one.ksplit || s.nw != one.nw)) wrong(nt, kt, M, "sums in another order than one row alone");
      }
  for (int nt = 1; nt <= 1024; ++nt)                        // half strips: every strip once, by the waves of the whole ones
    for (int kt : {63, 64, 128, 448}) {
      const int ns = strips_half(nt, kt, 9);
      const StripShape w = strip_shape(nt, kt, 9);
      if (!ns) continue;
      if (w.nw != w.ksplit || ns > w.nw || kt < 64 || strips_half(nt, kt, 17)) wrong(nt, kt, 9, "half strips by other waves");
      std::vector<int> seen(nt);
      for (int id = 0; id < half_grid(nt, ns); ++id)
        for (int i = 0; i < ns; ++i)
          if (half_strip_at(id, i, ns) < nt) seen[half_strip_at(id, i, ns)] += i < ns - 1 ? 2 : 1;
      for (int t = 0; t < nt; ++t)
        if (seen[t] != 2) wrong(nt, kt, t, "strip not covered once");
    }
  // loads that the waves of a block wait for: every tile of a stage once, and no wave outside the counts that the kernel's waits know
  for (auto f : {BlockPlace{16, 16}, BlockPlace{12, 16}, BlockPlace{8, 16}, BlockPlace{12, 12}, BlockPlace{8, 12}, BlockPlace{8, 8}})
    for (int used = 1; used <= f.row; ++used) {
      int n = 0;
      for (int w = 0; w < 8; ++w) {
        const int r = block_requests(w, f.col, used);
        n += r;
        if (w + 8 * (r - 1) >= f.col + used || w + 8 * r < f.col + used) wrong(f.col, f.row, used, "tile without a request, or a request without a tile");
        if (r < block_requests(7, f.col, 1) || r > block_requests(0, f.col, f.row)) wrong(f.col, f.row, used, "a count that no wait is for");
        if (used == f.row && r < block_requests(7, f.col, f.row)) wrong(f.col, f.row, used, "a count that no wait of a full block is for");
      }
      if (n != f.col + used) wrong(f.col, f.row, used, "requests");
    }
  for (int M = 1; M <= 4096; M += M % 16 == 1 ? 15 : 1)      // every block of a blocked launch exactly once
    for (int nt : {1, 16, 17, 128, 256, 384, 1546, 1792})
      for (auto f : {BlockPlace{16, 16}, BlockPlace{12, 16}, BlockPlace{8, 16}, BlockPlace{12, 12}, BlockPlace{8, 12}, BlockPlace{8, 8}}) {
        const BlockOrder o = block_order(nt, M, f.col, f.row);
        const int rblocks = ceil_div(M, 16 * f.row), cols = ceil_div(nt, f.col);
        std::vector<int> seen((size_t)rblocks * cols);
        int n = 0;
        for (int id = 0; id < 8 * o.share; ++id) {
          const BlockPlace p = block_place(o, id);
          if (p.col == -1) continue;
          ++n;
          if (p.col < 0 || p.col >= cols || p.row < 0 || p.row >= rblocks || seen[(size_t)p.row * cols + p.col]++) wrong(nt, f.col * 100 + f.row, M, "block out of place");
        }
        if (n != rblocks * cols) wrong(nt, f.col * 100 + f.row, M, "blocks missing");
      }
  return bad != 0;
}
